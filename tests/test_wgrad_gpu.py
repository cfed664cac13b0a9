"""Weight gradients on the bf16 matrix cores at the edges of their strips: every
conv's gradient against the FP64 oracle on frames that are narrower than a strip,
ragged in both directions, and with channel counts that leave a block of 16
or 32 partly empty or split over the two sources of a decoder's input."""
import numpy as np
import pytest
import torch

import oracle
from _helpers import rel_l2, to_dev
from paper_2202_05977_amd import synth

pytestmark = pytest.mark.gpu

# per-conv relative L2 of the training tests: gradients sum 10^3..10^5 fp32 terms
# of both signs after an fp32 forward pass
TOL_GRAD = 1e-4
ODD = synth.NetConfig(levels=2, channels=(48, 80), kernel_sizes=(3, 5))      # blocks of 32 across the sources at 80
# input gradients through a pool and a concatenation on the same activation, the
# blocks of 32 of the concatenations cut across their sources, M = 1
NEST = synth.NetConfig(levels=4, channels=(16, 48, 32, 16), kernel_sizes=(3,))
NARROW = synth.NetConfig(levels=1, channels=(16,), kernel_sizes=(3,))        # 16 channels, 2 outputs


@pytest.mark.parametrize("cfg,sizes", [(ODD, [(2, 2)]), (ODD, [(34, 66)] * 2), (ODD, [(10, 130), (66, 6)]),
                                       (NEST, [(24, 40), (16, 8), (24, 40)]),
                                       (NARROW, [(33, 31)]), (NARROW, [(70, 97)] * 2)])
def test_weight_gradients_against_oracle(cfg, sizes):
    from paper_2202_05977_amd import wskp
    blob = synth.make_weights(cfg, 8)
    host, frames, targets = [], [], []
    for i, (H, W) in enumerate(sizes):
        fr = synth.make_frame(60 + i, H, W)
        host.append(fr)
        f = to_dev(fr)
        f["out"] = torch.empty_like(f["radiance"])
        frames.append(f)
        targets.append(f["clean"])
    dn = wskp.Denoiser(cfg, blob, "fp32")
    grad = torch.full((blob.size,), float("nan"), dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    Hs, Ws = [s[0] for s in sizes], [s[1] for s in sizes]
    ws = torch.full((wskp.wskp_train_workspace_size(dn.h, Hs, Ws),), 0xff, dtype=torch.uint8, device="cuda")
    wskp.wskp_train_grads(dn.h, frames, targets, grad, loss, ws)
    g = grad.cpu().numpy().astype(np.float64)
    total = sum(h * w for h, w in sizes)
    ref = np.zeros(blob.size)
    for fr, (h, w) in zip(host, sizes):
        ref += oracle.train_grads(fr, fr["clean"], blob, cfg)[1] * (h * w / total)
    off = 0
    for name, ci, co in synth.conv_shapes(cfg):
        n = ci * co * 9 + co
        a, b = g[off:off + n], ref[off:off + n]
        assert np.all(np.isfinite(a)), name
        if np.linalg.norm(b) > 0:
            assert rel_l2(a, b) <= TOL_GRAD, name
        else:
            assert not a.any(), name
        off += n
    dn.close()


ONE = synth.NetConfig(levels=1, channels=(16,), kernel_sizes=(3, 5))


def _grads(cfg, blob, fr):
    from paper_2202_05977_amd import wskp
    H, W = fr["depth"].shape[:2]
    dn = wskp.Denoiser(cfg, blob, "fp32")
    f = to_dev(fr)
    f["out"] = torch.empty_like(f["radiance"])
    grad, loss = torch.empty(blob.size, device="cuda"), torch.empty(1, device="cuda")
    ws = torch.empty(wskp.wskp_train_workspace_size(dn.h, [H], [W]), dtype=torch.uint8, device="cuda")
    wskp.wskp_train_grads(dn.h, [f], [f["clean"]], grad, loss, ws)
    g = grad.cpu().numpy().astype(np.float64)
    dn.close()
    return g, oracle.train_grads(fr, fr["clean"], blob, cfg)[1]


def test_activations_beyond_the_largest_bf16():
    """A channel of 0 and 3.4e38, which would round to infinity in bf16: the head's
    gradient for it, and for the others, is finite and the oracle's."""
    blob = synth.make_weights(ONE, 4)
    w0, head = blob[:1440].reshape(16, 10, 3, 3), blob[1456:-4].reshape(4, 16, 3, 3)
    w0[0] = 0
    w0[0, 9, 1, 1] = 3.4e38
    blob[1440] = 0
    head[:, 0] = 0
    head[:, 0, 1, 1] = np.array([1, -1, 1, -1]) * 2.0 ** -125
    fr = synth.make_frame(5, 40, 70)
    fr["depth"][:] = np.where(fr["depth"] < np.median(fr["depth"]), 1.0, 10.0)
    g, ref = (v[1456:-4].reshape(4, 16, 9) for v in _grads(ONE, blob, fr))
    assert np.all(np.isfinite(g))
    assert rel_l2(g[:, 0], ref[:, 0]) <= TOL_GRAD and rel_l2(g[:, 1:], ref[:, 1:]) <= TOL_GRAD


@pytest.mark.parametrize("y,x", [(0, 0), (32, 44)])
def test_infinite_input_in_a_corner(y, x):
    """An infinite input where every activation that sees it is zero: the taps that
    pair it with such an activation are zero times infinity, the taps that would
    pair it with a pixel outside the image are the oracle's.  (32, 44): the last
    row of its strip and a column within one."""
    blob = synth.make_weights(ONE, 4)
    w0 = blob[:1440].reshape(16, 10, 3, 3)
    w0[:, 6] = -np.abs(w0[:, 6])
    fr = synth.make_frame(5, 33, 45)
    fr["normal"][y, x, 0] = np.inf
    g, ref = (v[:1440].reshape(16, 10, 9) for v in _grads(ONE, blob, fr))
    assert np.array_equal(np.isnan(g), np.isnan(ref)) and np.isnan(ref).sum() == 16 * 4
    fin = np.isfinite(ref)
    assert fin.sum() == 16 * 86 and rel_l2(g[fin], ref[fin]) <= TOL_GRAD


TWO = synth.NetConfig(levels=2, channels=(16, 32), kernel_sizes=(3, 5))


@pytest.mark.parametrize("cfg,sizes", [
    # 1040 32-row strips at level 0, 1040 16-row strips at level 1, each ending 4 and 2 rows into its
    # last; the input gradients of every kind on 8-row tiles (2064 of them at level 1)
    (TWO, [(2052, 4)] * 16),
    # 32-row strips of several columns, the last half a strip wide
    (TWO, [(180, 176)] * 16),
    # a forward pass on the split kernel
    (synth.SMALL, [(364, 364)]),
])
def test_large_batches_against_oracle(cfg, sizes):
    from paper_2202_05977_amd import wskp
    blob = synth.make_weights(cfg, 8)
    host = [synth.make_frame(80 + i % 2, H, W) for i, (H, W) in enumerate(sizes)]
    frames = []
    for fr in host:
        f = to_dev(fr)
        f["out"] = torch.empty_like(f["radiance"])
        frames.append(f)
    dn = wskp.Denoiser(cfg, blob, "fp32")
    grad, loss = torch.empty(blob.size, device="cuda"), torch.empty(1, device="cuda")
    ws = torch.empty(wskp.wskp_train_workspace_size(dn.h, [s[0] for s in sizes], [s[1] for s in sizes]),
                     dtype=torch.uint8, device="cuda")
    wskp.wskp_train_grads(dn.h, frames, [f["clean"] for f in frames], grad, loss, ws)
    g = grad.cpu().numpy().astype(np.float64)
    # (two distinct frames, so many times each)
    two = [oracle.train_grads(fr, fr["clean"], blob, cfg) for fr in host[:2]]
    ref = sum(t[1] for t in two) / len(two)
    assert abs(float(loss) - sum(t[0] for t in two) / len(two)) <= 1e-5 * float(loss)
    off = 0
    for name, ci, co in synth.conv_shapes(cfg):
        n = ci * co * 9 + co
        assert rel_l2(g[off:off + n], ref[off:off + n]) <= TOL_GRAD, name
        off += n
    dn.close()


def test_input_gradients_of_more_than_256_channels():
    """A decoder of 448 input channels.  Small weights and biases of one keep every
    pre-activation away from the ReLU's zero, on whose other side the rounding of a
    forward pass may put one of so few pixels."""
    cfg = synth.NetConfig(levels=2, channels=(192, 256), kernel_sizes=(3,))
    parts = []
    rng = np.random.default_rng(8)
    for name, ci, co in synth.conv_shapes(cfg):
        parts += [(0.05 * np.sqrt(2.0 / (9 * ci)) * rng.standard_normal(co * ci * 9)).astype(np.float32),
                  np.full(co, 0.0 if name == "head" else 1.0, np.float32)]
    g, ref = _grads(cfg, np.concatenate(parts), synth.make_frame(80, 24, 40))
    off = 0
    for name, ci, co in synth.conv_shapes(cfg):
        n = ci * co * 9 + co
        assert rel_l2(g[off:off + n], ref[off:off + n]) <= TOL_GRAD, name
        off += n


def test_split_weights_follow_an_adam_step():
    """A frame of the split kernel after a step equals, bit for bit, that of a new handle
    with the weights read back."""
    from paper_2202_05977_amd import wskp
    cfg = synth.SMALL
    blob = synth.make_weights(cfg, 8)
    dn = wskp.Denoiser(cfg, blob, "fp32")
    f = to_dev(synth.make_frame(9, 364, 364))
    before = dn(f).clone()
    n = blob.size
    g = torch.randn(n, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    wskp.wskp_adam(dn.h, g, torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda"), 1, lr=1e-3)
    w = torch.empty(n, device="cuda")
    wskp.wskp_get_weights(dn.h, w)
    new = wskp.Denoiser(cfg, w.cpu().numpy(), "fp32")
    after = dn(f)
    assert torch.equal(after, new(f)) and not torch.equal(after, before)
    dn.close()
    new.close()
