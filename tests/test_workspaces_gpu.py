"""Workspaces of exactly the size that the library asks for: nothing is written past
them, and they hold no more than what is written."""
import numpy as np
import pytest
import torch

from _helpers import to_dev
from paper_2202_05977_amd import synth

pytestmark = pytest.mark.gpu

GUARD = 4096


def _guarded(n):
    return torch.full((n + GUARD,), 0xa5, dtype=torch.uint8, device="cuda")


def _untouched(buf, n):
    return bool((buf[n:] == 0xa5).all())


@pytest.mark.parametrize("L", [2, 3, 4, 6])
def test_multiresolution_workspace(L):
    """The filtered image of every level; the pooled irradiance where levels past the
    first three are filtered from it.  256-byte regions."""
    from paper_2202_05977_amd import wskp
    cfg = synth.NetConfig(levels=1, channels=(16,), kernel_sizes=(3, 5))
    dn = wskp.Denoiser(cfg, np.zeros(synth.num_weights(cfg), np.float32), "fp32")
    h = dn.h
    H, W = 64, 96
    region = lambda l: ((H >> l) * (W >> l) * 12 + 255) // 256 * 256  # noqa: E731
    need = sum(region(l) for l in range(L)) + (sum(region(l) for l in range(1, L)) if L > 3 else 0)
    assert wskp.wskp_mr_workspace_size(h, L, H, W) == need
    rng = np.random.default_rng(L)
    d = lambda a: torch.from_numpy(a.astype(np.float32)).cuda()  # noqa: E731
    heads = [d(synth.make_head(40 + l, 1, H >> l, W >> l, 2)) for l in range(L)]
    alphas = [d(rng.uniform(0, 1, (H >> l, W >> l))) for l in range(L - 1)]
    c = d(rng.gamma(0.5, 2.0, (H, W, 3)))
    buf = _guarded(need)
    y = wskp.mr_reconstruct(h, heads, c, alphas, None, ws=buf[:need])
    assert torch.equal(y, wskp.mr_reconstruct(h, heads, c, alphas, None)) and _untouched(buf, need)
    dn.close()


@pytest.mark.parametrize("sizes", [[(64, 64)] * 3, [(40, 72), (64, 32)]])
def test_training_workspace(sizes):
    from paper_2202_05977_amd import wskp
    cfg = synth.HD
    dn = wskp.Denoiser(cfg, synth.make_weights(cfg, 3), "fp32")
    frames = []
    for i, (H, W) in enumerate(sizes):
        f = to_dev(synth.make_frame(70 + i, H, W))
        f["out"] = torch.empty_like(f["radiance"])
        frames.append(f)
    need = wskp.wskp_train_workspace_size(dn.h, [s[0] for s in sizes], [s[1] for s in sizes])
    grads = []
    for buf in (_guarded(need), torch.empty(2 * need, dtype=torch.uint8, device="cuda")):
        grad = torch.empty(synth.num_weights(cfg), device="cuda")
        ws = buf[:need] if buf.numel() == need + GUARD else buf
        wskp.wskp_train_grads(dn.h, frames, [f["clean"] for f in frames], grad, torch.empty(1, device="cuda"), ws)
        grads.append(grad)
        assert ws is buf or _untouched(buf, need)
    assert torch.equal(*grads) and bool(torch.isfinite(grads[0]).all())
    # 8 crops of 256x256: without room for the decoders' concatenated inputs (201 MB), which
    # the gradients read in place
    assert wskp.wskp_train_workspace_size(dn.h, [256] * 8, [256] * 8) < 800 << 20
    dn.close()
