"""FP8 convs at the edges of their tiles: a frame and a crop of it, whose tiles begin
and end elsewhere, hold the same values away from the crop's border, bit for bit."""
import numpy as np
import pytest
import torch

from _helpers import to_dev
from paper_2202_05977_amd import synth

pytestmark = pytest.mark.gpu

MARGIN = 8      # above the reach of a two-level net's last conv


@pytest.mark.parametrize("channels", [(32, 64), (96, 32), (128, 96)])
@pytest.mark.parametrize("crop", [(2, 60, 4, 70), (10, 52, 26, 92), (6, 64, 0, 34)])
def test_crop_holds_the_same_values(channels, crop):
    from paper_2202_05977_amd import wskp
    cfg = synth.NetConfig(levels=2, channels=channels, kernel_sizes=(3, 5, 7))
    dn = wskp.Denoiser(cfg, synth.make_weights(cfg, 2), "fp8", act_scales=np.array([1, 3, 2, 2], np.float32) / 448)
    y0, y1, x0, x1 = crop

    def maps(f):
        dn(f)
        torch.cuda.synchronize()
        H, W = f["radiance"].shape[:2]
        return [dn.intermediate([H], [W], 0, k).float().clone() for k in (0, 1, 100, 200)]

    full = to_dev(synth.make_frame(3, 64, 96))
    part = {k: v[y0:y1, x0:x1].contiguous() for k, v in full.items()}
    for name, a, b, l in zip(("e0", "e1", "u0", "head"), maps(full), maps(part), (0, 1, 0, 0)):
        a, m = a[y0 >> l:y1 >> l, x0 >> l:x1 >> l], MARGIN >> l
        assert torch.isfinite(a).all(), name
        assert torch.equal(a[m:-m, m:-m], b[m:-m, m:-m]), name
    dn.close()
