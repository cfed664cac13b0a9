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
