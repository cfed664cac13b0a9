"""The cut tiles of FP32 frames of few pixels: a frame on its own (two-row tiles of
one output block, five-row decode tiles) equals, bit for bit, the same frame inside
a batch that fills the GPU (full tiles)."""
import pytest
import torch

from _helpers import to_dev
from paper_2202_05977_amd import synth

pytestmark = pytest.mark.gpu

SMALL = synth.SMALL
WIDE = synth.NetConfig(levels=2, channels=(48, 80), kernel_sizes=(3, 11))    # 3 and 5 blocks, decode radius 5
EXP = synth.NetConfig(levels=2, channels=(64, 16), kernel_sizes=(5,), weight_act="exp")
REP = synth.NetConfig(levels=2, channels=(16, 32), kernel_sizes=(3, 5, 15), conv_size=5)


@pytest.mark.parametrize("cfg", [SMALL, WIDE, EXP, REP], ids=["small", "wide", "exp", "5x5"])
@pytest.mark.parametrize("size", [(4, 4), (20, 36), (100, 72)])
@pytest.mark.parametrize("graph", [False, True])
def test_small_frame_equals_itself_in_a_large_batch(cfg, size, graph):
    from paper_2202_05977_amd import wskp
    dn = wskp.Denoiser(cfg, synth.make_weights(cfg, 4), "fp32")
    small = to_dev(synth.make_frame(5, *size))
    one = dn(small)
    filler = to_dev(synth.make_frame(6, 256, 320))
    frames = [dict(f, out=torch.full_like(f["radiance"], float("nan"))) for f in [small] + [filler] * 24]
    for _ in range(2):
        dn.batch(frames, flags=wskp.BATCH_GRAPH if graph else 0)
    torch.cuda.synchronize()
    assert torch.isfinite(one).all()
    assert torch.equal(frames[0]["out"], one)
    assert torch.equal(frames[1]["out"], dn(filler)) and torch.equal(frames[24]["out"], frames[1]["out"])
    dn.close()
