"""Tensor-form decode with whole-record loads (any float alignment, odd and
largest kernel counts) and the multi-resolution reconstruction of 2..6 levels
in two launches against its steps one by one."""
import numpy as np
import pytest
import torch

import oracle
from _helpers import TOL_FP32, max_rel, rel_l2
from paper_2202_05977_amd import synth

pytestmark = pytest.mark.gpu


def _handle(ks):
    from paper_2202_05977_amd import wskp
    cfg = synth.NetConfig(levels=1, channels=(16,), kernel_sizes=ks)
    return wskp.Denoiser(cfg, np.zeros(synth.num_weights(cfg), np.float32), "fp32")


@pytest.mark.parametrize("ks,H,W", [((7,), 17, 33), ((3, 5, 7), 1, 1), ((3, 5, 7, 9, 11, 13, 15), 45, 70),
                                    ((1, 3, 5, 7, 9, 11, 13, 15), 31, 97)])
def test_records_of_any_float_alignment(ks, H, W):
    from paper_2202_05977_amd import wskp
    dn, M = _handle(ks), len(ks)
    head = synth.make_head(1, 2, H, W, M)
    rng = np.random.default_rng(2)
    c = rng.uniform(0.1, 2.0, (2, H, W, 3)).astype(np.float32)
    mod = rng.uniform(0.1, 1.0, (2, H, W, 3)).astype(np.float32)

    def shifted(a, k):   # the same values k floats past a 16-byte boundary
        buf = torch.empty(a.size + 4, dtype=torch.float32, device="cuda")
        buf[k:k + a.size] = torch.from_numpy(a.ravel()).cuda()
        return buf[k:k + a.size].view(a.shape)

    ref = np.stack([oracle.decode(head[n], c[n], mod[n], ks) for n in range(2)])
    outs = []
    for k in (0, 1, 3):
        out = torch.full((2, H, W, 3), float("nan"), device="cuda")
        wskp.wskp_decode(dn.h, shifted(head, k), shifted(c, k), shifted(mod, k), out)
        outs.append(out)
    y = outs[0].cpu().numpy()
    assert rel_l2(y, ref) <= TOL_FP32 and max_rel(y, ref) <= TOL_FP32
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    dn.close()


@pytest.mark.parametrize("L,H,W", [(2, 2, 2), (2, 66, 130), (3, 4, 4), (3, 100, 68), (4, 72, 104), (5, 80, 48), (6, 96, 160)])
@pytest.mark.parametrize("remodulate", [False, True])
def test_levels_in_one_launch_equal_the_steps(L, H, W, remodulate):
    from paper_2202_05977_amd import wskp
    ks = (3, 5, 7)
    dn = _handle(ks)
    g = torch.Generator("cuda").manual_seed(3)
    c = torch.rand((H, W, 3), device="cuda", generator=g) + 0.1
    mod = torch.rand((H, W, 3), device="cuda", generator=g) if remodulate else None
    heads = [torch.from_numpy(synth.make_head(4 + l, 1, H >> l, W >> l, 3)).cuda() for l in range(L)]
    alphas = [torch.rand((H >> l, W >> l), device="cuda", generator=g) for l in range(L - 1)]
    got = wskp.mr_reconstruct(dn.h, heads, c, alphas, mod)
    cs, fs = [c], []
    for l in range(1, L):
        p = torch.empty((H >> l, W >> l, 3), device="cuda")
        wskp.wskp_pool2(dn.h, cs[-1], p)
        cs.append(p)
    for l in range(L):
        f = torch.empty((1, H >> l, W >> l, 3), device="cuda")
        wskp.wskp_decode(dn.h, heads[l], cs[l][None].contiguous(), None, f)
        fs.append(f[0])
    o = fs[-1]
    for l in range(L - 2, -1, -1):
        n = torch.empty_like(fs[l])
        wskp.wskp_mr_blend(dn.h, fs[l], o, alphas[l], mod if l == 0 else None, n)
        o = n
    assert torch.equal(got, o)
    dn.close()
