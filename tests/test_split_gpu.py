"""FP32 3x3 convs as six bf16 MFMAs (frames of at least 2^17 pixels): parity
with the FP64 oracle at the edges of its tiles and of its range, non-finite
inputs, and batches of frames on both sides of the size rule."""
import numpy as np
import pytest
import torch

import oracle
from _helpers import TOL_FP32, max_rel, rel_l2, to_dev
from paper_2202_05977_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg_name,H,W", [
    ("small", 8, 16384),      # exactly 2^17 pixels, one 8-row tile of rows
    ("small", 364, 364),      # 4 rows and 12 columns past the last whole tile
    ("small", 10924, 12),     # less than a tile wide
    ("hd", 360, 376),         # three and four groups of 32 channels, 4-row tiles on the coarse levels
])
def test_split_convs_against_oracle(cfg_name, H, W):
    from paper_2202_05977_amd import wskp
    cfg = synth.CONFIGS[cfg_name]
    blob = synth.make_weights(cfg, 4)
    fr = synth.make_frame(5, H, W)
    dn = wskp.Denoiser(cfg, blob, "fp32")
    y = dn(to_dev(fr)).cpu().numpy()
    ref = oracle.denoise(fr, blob, cfg)
    assert H * W >= 1 << 17
    assert rel_l2(y, ref) <= TOL_FP32 and max_rel(y, ref) <= TOL_FP32
    dn.close()


def test_split_convs_with_nonfinite_inputs():
    """An infinite and a NaN albedo, and an infinite normal: the same outputs
    are finite as with plain fp32 sums, and those agree."""
    from paper_2202_05977_amd import wskp
    cfg = synth.SMALL
    blob = synth.make_weights(cfg, 4)
    H, W = 364, 364
    fr = synth.make_frame(6, H, W)
    fr["albedo"][40, 50, 1] = np.inf
    fr["albedo"][200, 300, 0] = np.nan
    fr["normal"][300, 31, 2] = -np.inf
    fr["normal"][100, 200, 0] = 3.4e38
    # the same rows and columns in a frame small enough for the fp32 MFMAs
    # (cropped well outside the net's and the filter's reach of the pixels)
    dn = wskp.Denoiser(cfg, blob, "fp32")
    y = dn(to_dev(fr)).cpu().numpy()
    for cy, cx in ((40, 50), (200, 300), (300, 31), (100, 200)):
        y0, x0 = max(0, cy // 4 * 4 - 60), max(0, cx // 4 * 4 - 60)
        crop = {k: np.ascontiguousarray(v[y0:y0 + 124, x0:x0 + 124]) for k, v in fr.items()}
        h, w = crop["depth"].shape[:2]
        z = dn(to_dev(crop)).cpu().numpy()
        # compare away from the crop's own borders
        iy, ix = slice(28 if y0 else 0, h - 28), slice(28 if x0 else 0, w - 28)
        a, b = y[y0:y0 + h, x0:x0 + w][iy, ix], z[iy, ix]
        fin = np.isfinite(b)
        assert np.array_equal(fin, np.isfinite(a)), (cy, cx)
        assert rel_l2(a[fin], b[fin]) <= TOL_FP32, (cy, cx)
    dn.close()


@pytest.mark.parametrize("graph", [False, True])
def test_batch_across_the_size_rule_equals_single_frames(graph):
    from paper_2202_05977_amd import wskp
    cfg = synth.SMALL
    dn = wskp.Denoiser(cfg, synth.make_weights(cfg, 4), "fp32")
    for sizes in ([(364, 364), (64, 96), (480, 640), (124, 36)], [(480, 640), (364, 364)], [(64, 96), (364, 364)]):
        frames = []
        for i, (H, W) in enumerate(sizes):
            f = to_dev(synth.make_frame(20 + i, H, W))
            f["out"] = torch.full_like(f["radiance"], float("nan"))
            frames.append(f)
        dn.batch(frames, wskp.BATCH_GRAPH if graph else 0)
        torch.cuda.synchronize()
        got = [f["out"].clone() for f in frames]
        for g, f in zip(got, frames):
            assert torch.equal(g, dn(f))
    dn.close()


def _time(run, n=7):
    """Median time of a pass, milliseconds."""
    run()
    t = []
    for _ in range(n):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        run()
        b.record()
        b.synchronize()
        t.append(a.elapsed_time(b))
    return sorted(t)[n // 2]


def test_split_convs_over_the_whole_range():
    """Weights and activations beyond the largest bf16 (3.39e38), which round to
    infinity there: the first conv passes depth (0 or 1) on times 3.4e38, the head takes
    2^-125 of it, beside ordinary channels."""
    from paper_2202_05977_amd import wskp
    cfg = synth.NetConfig(levels=1, channels=(32,), kernel_sizes=(3, 5))
    blob = synth.make_weights(cfg, 4)
    w0, head = blob[:32 * 90].reshape(32, 10, 3, 3), blob[32 * 90 + 32:-4].reshape(4, 32, 3, 3)
    w0[0] = 0
    w0[0, 9, 1, 1] = 3.4e38
    blob[32 * 90] = 0
    head[:, 0] = 0
    head[:, 0, 1, 1] = np.array([1, -1, 1, -1]) * 2.0 ** -125
    fr = synth.make_frame(5, 364, 364)
    fr["depth"][:] = np.where(fr["depth"] < np.median(fr["depth"]), 1.0, 10.0)
    dn = wskp.Denoiser(cfg, blob, "fp32")
    y = dn(to_dev(fr)).cpu().numpy()
    e0 = dn.intermediate([364], [364], 0, 0)[..., 0].cpu().numpy()
    assert np.array_equal(e0, np.where(fr["depth"][..., 0] > 5, np.float32(3.4e38), np.float32(0)))
    ref = oracle.denoise(fr, blob, cfg)
    assert rel_l2(y, ref) <= TOL_FP32 and max_rel(y, ref) <= TOL_FP32
    dn.close()


def test_nan_background_takes_no_longer():
    """Every output of the first conv under NaN normals is NaN; half a frame of them
    costs what any frame costs (1.5: the spread of a short run)."""
    from paper_2202_05977_amd import wskp
    dn = wskp.Denoiser(synth.SMALL, synth.make_weights(synth.SMALL, 4), "fp32")
    f = to_dev(synth.make_frame(7, 512, 512))
    clean = _time(lambda: dn(f))
    f["normal"][:256] = float("nan")
    assert _time(lambda: dn(f)) <= 1.5 * clean
    dn.close()


def test_nan_gradients_take_no_longer():
    """A training step whose loss is NaN: every input gradient is."""
    from paper_2202_05977_amd import wskp
    cfg = synth.SMALL
    dn = wskp.Denoiser(cfg, synth.make_weights(cfg, 4), "fp32")
    f = to_dev(synth.make_frame(7, 64, 64))
    f["out"] = torch.empty_like(f["radiance"])
    target = f["clean"].clone()
    grad, loss = torch.empty(synth.num_weights(cfg), device="cuda"), torch.empty(1, device="cuda")
    ws = torch.empty(wskp.wskp_train_workspace_size(dn.h, [64], [64]), dtype=torch.uint8, device="cuda")
    step = lambda: wskp.wskp_train_grads(dn.h, [f], [target], grad, loss, ws)  # noqa: E731
    clean = _time(step)
    target.fill_(float("nan"))
    t = _time(step)
    assert bool(torch.isnan(grad).any()) and t <= 1.5 * clean
    dn.close()


@pytest.mark.parametrize("channels,split", [((16,), False), ((16, 16, 16), False), ((16, 64), False), ((16, 256), True),
                                            ((32, 16), True)])
def test_nets_of_narrow_layers_keep_the_fp32_mfmas(channels, split):
    """A layer's values do not depend on the frame's tiling, so those of a net that
    runs one kernel at all sizes are, away from the borders, bitwise those of a
    small frame cut out of it."""
    from paper_2202_05977_amd import wskp
    cfg = synth.NetConfig(levels=len(channels), channels=channels, kernel_sizes=(3, 5))
    dn = wskp.Denoiser(cfg, synth.make_weights(cfg, 4), "fp32")
    fr = synth.make_frame(5, 364, 364)
    dn(to_dev(fr))
    a = dn.intermediate([364], [364], 0, 200)[100:228, 120:248].clone()
    dn(to_dev({k: np.ascontiguousarray(v[100:228, 120:248]) for k, v in fr.items()}))
    b = dn.intermediate([128], [128], 0, 200)
    same = torch.equal(a[24:-24, 24:-24], b[24:-24, 24:-24])
    assert same == (not split)
    dn.close()
