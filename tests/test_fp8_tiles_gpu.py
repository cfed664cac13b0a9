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


@pytest.mark.parametrize("channels", [(32, 64), (64, 128), (96, 32)])
def test_small_frame_on_short_tiles_holds_the_values_of_a_large_one(channels):
    """A frame of 900 8-row tiles and crops of it small enough for 4-row tiles, on both
    sides of 256 8-row tiles."""
    from paper_2202_05977_amd import wskp
    cfg = synth.NetConfig(levels=2, channels=channels, kernel_sizes=(3, 5, 7))
    dn = wskp.Denoiser(cfg, synth.make_weights(cfg, 2), "fp8", act_scales=np.array([1, 3, 2, 2], np.float32) / 448)
    full = to_dev(synth.make_frame(3, 480, 480))

    def maps(f):
        dn(f)
        torch.cuda.synchronize()
        H, W = f["radiance"].shape[:2]
        return [dn.intermediate([H], [W], 0, k).float().clone() for k in (0, 1, 100, 200)]

    whole = maps(full)
    for h, w in ((256, 256), (264, 256), (62, 90)):
        part = {k: v[10:10 + h, 36:36 + w].contiguous() for k, v in full.items()}
        for name, a, b, l in zip(("e0", "e1", "u0", "head"), whole, maps(part), (0, 1, 0, 0)):
            a, m = a[10 >> l:10 + h >> l, 36 >> l:36 + w >> l], MARGIN >> l
            assert torch.equal(a[m:-m, m:-m], b[m:-m, m:-m]), (name, h, w)
    dn.close()
