"""Every pass of the frame decode writes the same image, bit for bit."""
import pytest
import torch

from _helpers import to_dev
from paper_2202_05977_amd import synth

pytestmark = pytest.mark.gpu

CFG = synth.NetConfig(levels=2, channels=(16, 32), kernel_sizes=(3, 5, 15), conv_size=5)


def test_tall_tile_rows_are_stored_once():
    """Radius 7 has 39-row decode tiles, whose last run of five rows overlaps the one
    above: every pass writes the same image."""
    from paper_2202_05977_amd import wskp
    dn = wskp.Denoiser(CFG, synth.make_weights(CFG, 4), "fp32")
    f = to_dev(synth.make_frame(6, 256, 320))
    first = dn(f)
    for _ in range(8):
        assert torch.equal(dn(f), first)
    dn.close()
