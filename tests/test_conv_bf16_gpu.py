"""bf16 convs on 32x32x16 MFMAs at the edges of their tiles: every layer of a
net against the FP64 oracle on the stored (bf16) inputs, for 4-, 8- and 12-row
tiles and ragged frames, 3x3 and 5x5."""
import numpy as np
import pytest
import torch

import oracle
from _helpers import TOL_BF16, TOL_BF16_MAX, max_rel, rel_l2, to_dev
from paper_2202_05977_amd import synth

pytestmark = pytest.mark.gpu

THREE = synth.NetConfig(levels=3, channels=(32, 64, 96), kernel_sizes=(3, 5, 7))
THREE5 = synth.NetConfig(levels=3, channels=(32, 64, 32), kernel_sizes=(3, 5, 7), conv_size=5)


@pytest.mark.parametrize("cfg,sizes", [
    (THREE, [(36, 44)]),                     # 4-row tiles, one row and 12 columns past them
    (THREE, [(4, 4)]),                       # a level of one pixel
    (THREE, [(132, 100), (4, 300), (68, 8)]),
    (THREE, [(1092, 1924)] * 2),             # 12-row tiles: 2 x 61 x 91 of them, ragged on both sides
    (THREE5, [(68, 100)]),
    (THREE5, [(260, 516), (8, 8)]),
])
def test_decoder_layers_against_oracle(cfg, sizes):
    """u_l = relu(conv([up(u_{l+1}), e_l])) of the stored maps, to the rounding
    of the output: 2^-8 of its value plus the fp32 sum's error."""
    from paper_2202_05977_amd import wskp
    blob = synth.make_weights(cfg, 6)
    dn = wskp.Denoiser(cfg, blob, "bf16")
    frames = []
    for i, (H, W) in enumerate(sizes):
        f = to_dev(synth.make_frame(30 + i, H, W))
        f["out"] = torch.full_like(f["radiance"], float("nan"))
        frames.append(f)
    dn.batch(frames)
    torch.cuda.synchronize()
    Hs, Ws = [s[0] for s in sizes], [s[1] for s in sizes]
    shapes, k, off, convs = synth.conv_shapes(cfg), cfg.conv_size, 0, {}
    for name, ci, co in shapes:
        w = torch.from_numpy(blob[off:off + co * ci * k * k].reshape(co, ci, k, k)).cuda().bfloat16().double()
        b = torch.from_numpy(blob[off + co * ci * k * k:off + co * ci * k * k + co]).cuda().double()
        convs[name] = (w, b)
        off += co * ci * k * k + co

    def conv(x, name):
        w, b = convs[name]
        r = k // 2
        H, W = x.shape[:2]
        xp = torch.nn.functional.pad(x, (0, 0, r, r, r, r))
        y = b.expand(H, W, -1)
        for dy in range(k):
            for dx in range(k):
                y = y + xp[dy:dy + H, dx:dx + W] @ w[:, :, dy, dx].t()
        return torch.relu(y)

    for f in range(len(sizes)):
        get = lambda which: dn.intermediate(Hs, Ws, f, which).double()  # noqa: E731
        L = cfg.levels
        pairs = [(conv(get(300 + l - 1), f"enc{l}"), get(l), f"enc{l}") for l in range(1, L)]
        for l in range(L - 2, -1, -1):
            up = get(100 + l + 1).repeat_interleave(2, 0).repeat_interleave(2, 1)
            pairs.append((conv(torch.cat([up, get(l)], -1), f"dec{l}"), get(100 + l), f"dec{l}"))
        for ref, got, name in pairs:
            tol = 2.0 ** -8 * ref.abs() + 1e-5 * float(ref.abs().max())
            assert bool(((got - ref).abs() <= tol).all()), (name, f)
        for l in range(L - 1):   # the 2x2 means of the stored values, bitwise
            e = dn.intermediate(Hs, Ws, f, l).float()
            m = 0.25 * (((e[0::2, 0::2] + e[0::2, 1::2]) + e[1::2, 0::2]) + e[1::2, 1::2])
            assert torch.equal(dn.intermediate(Hs, Ws, f, 300 + l), m.bfloat16()), (l, f)
    fr = synth.make_frame(30, *sizes[0])
    if sizes[0][0] * sizes[0][1] < 1 << 18:
        y = frames[0]["out"].cpu().numpy()
        ref = oracle.denoise(fr, blob, cfg)
        assert rel_l2(y, ref) <= TOL_BF16 and max_rel(y, ref) <= TOL_BF16_MAX
    assert all(bool(torch.isfinite(f["out"]).all()) for f in frames)
    dn.close()


@pytest.mark.parametrize("k", [3, 5])
@pytest.mark.parametrize("block", [(1.0, 2.0 ** -8 - 2.0 ** -16, 2.0 ** -16 - 2.0 ** -24, 1.5 * 2.0 ** -24),
                                   (1.0, 2.0 ** -8 - 2.0 ** -16, 1.5 * 2.0 ** -24, 2.0 ** -16 - 2.0 ** -24)])
def test_pooled_means_add_in_order(block, k):
    """Blocks whose sum is a bf16 tie's upper or lower side depending on which value
    of the second row is added first: level 1's means are of the sums in the order
    (0,0), (0,1), (1,0), (1,1).  Both encoders copy the albedo's first channel."""
    from paper_2202_05977_amd import wskp
    cfg = synth.NetConfig(levels=3, channels=(32, 32, 32), kernel_sizes=(3,), conv_size=k)
    parts = []
    for name, ci, co in synth.conv_shapes(cfg):
        w = np.zeros((co, ci, k, k), np.float32)
        if name == "enc0":
            w[:, 3, k // 2, k // 2] = 1.0
        elif name == "enc1":
            w[np.arange(32), np.arange(32), k // 2, k // 2] = 1.0
        parts += [w.ravel(), np.zeros(co, np.float32)]
    dn = wskp.Denoiser(cfg, np.concatenate(parts), "bf16")
    H, W = 24, 152
    fr = synth.make_frame(3, H, W)
    v = np.tile(np.array(block, np.float32).reshape(2, 2), (H // 4, W // 4))     # level 1's map
    fr["albedo"][:] = np.repeat(np.repeat(v, 2, 0), 2, 1)[..., None]
    dn(to_dev(fr))
    e1 = dn.intermediate([H], [W], 0, 1).float().cpu()
    assert torch.equal(e1, torch.from_numpy(v)[..., None].expand_as(e1))
    s = np.float32(block[0])
    for b in block[1:]:
        s = np.float32(s + np.float32(b))
    mean = torch.tensor(0.25 * s, dtype=torch.float32).bfloat16()
    p1 = dn.intermediate([H], [W], 0, 301).cpu()
    assert torch.equal(p1, mean.expand_as(p1))
    dn.close()
