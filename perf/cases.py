"""The workloads whose speed is watched, each through the public entry points.

``listed()`` names them, ``draw(rng)`` gives more of the same ranges,
``prepare(case, seed)`` makes what a program has in hand before the call (the
frames on the device, the handle with its weights, the workspaces),
``run(state)`` is one pass, ``work(case)`` the bytes and operations that pass
cannot do without, and ``exact(case, seed)`` what it returns, evaluated in
float64 with plain torch.

Inputs have the distributions of ``paper_2202_05977_amd.synth`` (1-spp-like
noise with fireflies, Voronoi albedo, smooth normals and depth, He-normal
weights), drawn on the device so that a new state is quick to make.
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_2202_05977_amd import synth, wskp

DEV = "cuda"

# levels, widths, kernel sizes, weight activation and conv size of the
# networks (synth.SMALL, HD, PAPER6, REPVGG)
NETS = {
    "small": (3, (16, 32, 64), (3, 5, 7), "softplus", 3),
    "hd": (4, (32, 64, 96, 128), (3, 5, 7, 9, 11), "softplus", 3),
    "paper6": (4, (32, 64, 96, 128), (3, 5, 7, 9, 11, 13), "exp", 3),
    "repvgg": (4, (32, 64, 96, 128), (3, 5, 7, 9, 11), "softplus", 5),
}
EPS_NORM, EPS_ALBEDO, GAMMA, NEAR, FAR, EPS_SMAPE = 1e-10, 1e-3, 2.2, 1.0, 10.0, 0.01
STEP, LR, BETA1, BETA2, ADAM_EPS = 100, 1e-3, 0.9, 0.999, 1e-8


def listed():
    return [
        # the small net at its own frame size: seven short launches, where
        # launch latency and few workgroups count
        {"name": "denoise_small_fp32_128", "kind": "denoise", "net": "small", "prec": "fp32", "sizes": "128x128"},
        # the headline: one 720p frame, bf16 convolutions
        {"name": "denoise_hd_bf16_720p", "kind": "denoise", "net": "hd", "prec": "bf16", "sizes": "720x1280"},
        # the same frame at full precision (offline frames, references)
        {"name": "denoise_hd_fp32_720p", "kind": "denoise", "net": "hd", "prec": "fp32", "sizes": "720x1280"},
        # the fp8 form, at the size of the precision sweep
        {"name": "denoise_hd_fp8_1080p", "kind": "denoise", "net": "hd", "prec": "fp8", "sizes": "1080x1920"},
        # RepVGG blocks: every conv 5x5
        {"name": "denoise_repvgg_bf16_720p", "kind": "denoise", "net": "repvgg", "prec": "bf16", "sizes": "720x1280"},
        # the paper's kernel set with exp weights, a small frame that no tile size divides
        {"name": "denoise_paper6_bf16_ragged", "kind": "denoise", "net": "paper6", "prec": "bf16", "sizes": "376x664"},
        # one serving batch: a frame of each served resolution in one call
        {"name": "batch_hd_bf16_serving", "kind": "batch", "net": "hd", "prec": "bf16",
         "sizes": "360x640,720x1280,1080x1920,1440x2560"},
        # one training step of the network in the middle of a run (its Adam moments are in hand): 8 crops, fp32
        {"name": "train_hd_8x256", "kind": "train", "net": "hd", "prec": "fp32", "sizes": ",".join(["256x256"] * 8)},
        # decode and its adjoint alone, under autograd (a caller's own network in front)
        {"name": "decode_grad_8x256", "kind": "decode_grad", "n": 8, "h": 256, "w": 256, "kernels": "3,5,7,9,11"},
        # decode alone with the paper's six sizes, an odd frame just under 720p
        {"name": "decode_m6_odd", "kind": "decode", "n": 1, "h": 715, "w": 1273, "kernels": "3,5,7,9,11,13"},
        # temporal accumulation in front of the denoiser, one moving 720p frame
        {"name": "temporal_720p", "kind": "temporal", "h": 720, "w": 1280},
        # multi-resolution reconstruction, three levels of two sizes
        {"name": "mr_720p", "kind": "mr", "h": 720, "w": 1280, "levels": 3, "kernels": "3,5"},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _size(rng, area_lo, area_hi, align):
    """A frame of log-uniform area and an aspect ratio of 0.5 to 2.2, sides multiples of ``align``."""
    area, aspect = _log(rng, area_lo, area_hi), _log(rng, 0.5, 2.2)
    w = max(align, int(math.sqrt(area * aspect)) // align * align)
    h = max(align, int(area / w) // align * align)
    return h, w


def draw(rng):
    kind = rng.choice(["denoise", "denoise", "denoise", "batch", "train", "decode_grad", "decode", "temporal", "mr"])
    if kind in ("denoise", "batch"):
        net, prec = rng.choice([("small", "fp32"), ("small", "bf16"), ("hd", "bf16"), ("hd", "bf16"), ("hd", "fp32"),
                                ("hd", "fp8"), ("paper6", "bf16"), ("paper6", "fp32"), ("repvgg", "bf16"),
                                ("repvgg", "fp32")])
        # frames from 128x128 to 2560x1440 (bf16), 720p (fp32), less for 5x5 convs
        top = 9.2e5 if prec == "fp32" else 3.6e6
        top *= 0.4 if net == "repvgg" else 1.0
        align = 1 << (NETS[net][0] - 1)
        n = 1 if kind == "denoise" else rng.randint(2, 6)
        sizes = [_size(rng, 1.6e4, top / n if prec == "fp32" else top, align) for _ in range(n)]
        return {"kind": kind, "net": net, "prec": prec, "sizes": ",".join("%dx%d" % s for s in sizes)}
    if kind == "train":
        n = rng.randint(3, 8)
        one = _size(rng, 2e4, 6.5e4, 8)
        sizes = [one] * n if rng.random() < 0.7 else [_size(rng, 2e4, 3.3e4, 8) for _ in range(n)]
        return {"kind": "train", "net": "hd", "prec": "fp32", "sizes": ",".join("%dx%d" % s for s in sizes)}
    if kind == "decode_grad":
        n = rng.randint(1, 8)
        h, w = _size(rng, 4e3, 1.2e5, 1)
        m = rng.randint(1, 6)
        return {"kind": kind, "n": n, "h": h, "w": w, "kernels": ",".join(str(3 + 2 * i) for i in range(m))}
    if kind == "decode":
        h, w = _size(rng, 1e4, 9.2e5, 1)
        m = rng.randint(1, 6)
        first = rng.choice([3, 3, 1])
        return {"kind": kind, "n": rng.randint(1, 2), "h": h, "w": w,
                "kernels": ",".join(str(first + 2 * i) for i in range(m))}
    if kind == "temporal":
        h, w = _size(rng, 1.6e4, 2.1e6, 1)
        return {"kind": kind, "h": h, "w": w}
    levels = rng.randint(2, 4)
    h, w = _size(rng, 3e4, 9.2e5, 1 << (levels - 1))
    return {"kind": "mr", "h": h, "w": w, "levels": levels, "kernels": rng.choice(["3,5", "3,5,7", "5"])}


# ---------------------------------------------------------------- inputs
def _sizes(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["sizes"].split(",")]


def _kernels(case):
    return tuple(int(k) for k in case["kernels"].split(","))


def _gen(seed):
    g = torch.Generator(DEV)
    g.manual_seed(seed & 0x7FFFFFFFFFFF)
    return g


def _grid(h, w):
    x = torch.arange(w, device=DEV, dtype=torch.float64) + 0.5
    y = torch.arange(h, device=DEV, dtype=torch.float64) + 0.5
    return x[None, :], y[:, None]


def _scene(rng, h, w, shift=(0.0, 0.0)):
    """Irradiance, albedo, normal and depth of a procedural scene, seen from a camera moved by ``shift`` pixels."""
    x, y = _grid(h, w)
    px, py = x + shift[0], y + shift[1]
    u, v = px / w, py / h
    E = torch.full((h, w), 0.25, device=DEV, dtype=torch.float64)
    for a, fx, fy, ph in zip(rng.uniform(0.02, 0.12, 8), rng.uniform(-12, 12, 8), rng.uniform(-12, 12, 8),
                             rng.uniform(0, 2 * np.pi, 8)):
        E += a * (1.0 + torch.sin(2 * np.pi * (fx * u + fy * v) + ph))
    tint = torch.tensor(rng.uniform(0.8, 1.2, 3), device=DEV)
    sites, colours = rng.uniform(0, 1, (12, 2)), torch.tensor(rng.uniform(0.1, 0.9, (12, 3)), device=DEV)
    dist = torch.stack([(px - s[0] * w) ** 2 + (py - s[1] * h) ** 2 for s in sites])
    albedo = colours[dist.argmin(0)]
    hx, hy = torch.zeros_like(E), torch.zeros_like(E)
    for b, gx, gy, ps in zip(rng.uniform(0.005, 0.02, 4), rng.uniform(-6, 6, 4), rng.uniform(-6, 6, 4),
                             rng.uniform(0, 2 * np.pi, 4)):
        c = b * torch.cos(2 * np.pi * (gx * u + gy * v) + ps) * 2 * np.pi
        hx += c * gx
        hy += c * gy
    normal = torch.stack([-hx, -hy, torch.ones_like(hx)], -1)
    normal = normal / normal.norm(dim=-1, keepdim=True)
    s, t = rng.uniform(1, 4, 2), rng.uniform(0, 2 * np.pi, 2)
    d = 0.5 + 0.25 * (torch.sin(2 * np.pi * u * s[0] + t[0]) + torch.sin(2 * np.pi * v * s[1] + t[1]))
    return albedo * tint * E[..., None], albedo, normal, (1.0 + 9.0 * d.clamp(0, 1))[..., None]


def _noisy(clean, g):
    """1-spp noise: Gamma(1/2, 2) per channel (a squared normal) and 0.1 % fireflies 50 times as bright."""
    h, w, _ = clean.shape
    n = torch.randn((h, w, 3), device=DEV, generator=g).double().square()
    fire = torch.rand((h, w, 1), device=DEV, generator=g) < 1e-3
    return clean * torch.where(fire, 50.0 * n, n)


def _frame(seed, h, w):
    clean, albedo, normal, depth = _scene(np.random.default_rng(seed), h, w)
    f = {"radiance": _noisy(clean, _gen(seed)), "albedo": albedo, "normal": normal, "depth": depth, "clean": clean}
    return {k: v.float().contiguous() for k, v in f.items()}


def _frames(case, seed):
    return [_frame(1000 * seed + i, h, w) for i, (h, w) in enumerate(_sizes(case))]


def _convs(net):
    levels, ch, kernels, _, k = NETS[net]
    dims = [(10, ch[0])] + [(ch[l - 1], ch[l]) for l in range(1, levels)]
    dims += [(ch[l + 1] + ch[l], ch[l]) for l in range(levels - 2, -1, -1)]
    return dims + [(ch[0], 2 * len(kernels))], k


def _weights(net, seed):
    dims, k = _convs(net)
    rng = np.random.default_rng(seed + 77)
    parts = []
    for ci, co in dims:
        parts += [rng.standard_normal(co * ci * k * k, np.float32) * np.float32(math.sqrt(2.0 / (k * k * ci))),
                  rng.uniform(-0.05, 0.05, co).astype(np.float32)]
    return np.concatenate(parts)


def _moments(net, seed):
    """Adam's moments some steps into a run (gradients of the default initialisation are 1e-4 to 6e-4 a value)."""
    n, g = _weights(net, seed).size, _gen(seed + 31)
    m = 3e-4 * torch.randn(n, device=DEV, generator=g)
    return m, (3e-4) ** 2 * (0.5 + torch.rand(n, device=DEV, generator=g))


def _config(net):
    levels, ch, kernels, act, k = NETS[net]
    return synth.NetConfig(levels=levels, channels=ch, kernel_sizes=kernels, weight_act=act, conv_size=k,
                           eps_norm=EPS_NORM, eps_albedo=EPS_ALBEDO, gamma=GAMMA, depth_near=NEAR, depth_far=FAR)


def _decode_handle(kernels):
    """A handle for decode calls alone: its own network is not run."""
    cfg = synth.NetConfig(levels=1, channels=(16,), kernel_sizes=kernels, eps_norm=EPS_NORM)
    return wskp.Denoiser(cfg, np.zeros(synth.num_weights(cfg), np.float32), "fp32")


def _head(g, n, h, w, m):
    """Log-normal weights, then N(0, 1) logits."""
    x = torch.randn((n, h, w, 2 * m), device=DEV, generator=g)
    x[..., :m] = x[..., :m].exp()
    return x


def _decode_inputs(case, seed):
    g, n, h, w = _gen(seed), case["n"], case["h"], case["w"]
    frames = [_frame(1000 * seed + i, h, w) for i in range(n)]
    mod = torch.stack([f["albedo"] for f in frames]) + EPS_ALBEDO
    c = torch.stack([f["radiance"] for f in frames]) / mod
    head = _head(g, n, h, w, len(_kernels(case)))
    return head, c, mod, torch.randn((n, h, w, 3), device=DEV, generator=g) / (3 * n * h * w)


def _temporal_inputs(case, seed):
    """A panning camera and a disk that moves over the scene; the previous frame's accumulated radiance and lengths."""
    h, w = case["h"], case["w"]
    pan, vel, g = (1.37, -0.61), (2.3, 1.1), _gen(seed)
    out = []
    x, y = _grid(h, w)
    for t in (3, 4):
        clean, _, normal, depth = _scene(np.random.default_rng(seed), h, w, (t * pan[0], t * pan[1]))
        cx, cy = 0.3 * w + t * vel[0], 0.4 * h + t * vel[1]
        disk = ((x - cx) ** 2 + (y - cy) ** 2 <= (0.12 * min(h, w)) ** 2)[..., None]
        zero = torch.zeros((h, w), device=DEV, dtype=torch.float64)
        wpos = torch.stack([(x + t * pan[0]) / 1000.0 + zero, (y + t * pan[1]) / 1000.0 + zero, depth[..., 0] / 100.0], -1)
        on = torch.stack([(x - cx + 0.3 * w + t * vel[0]) / 1000.0 + zero,
                          (y - cy + 0.4 * h + t * vel[1]) / 1000.0 + zero, zero + 0.012], -1)
        up = torch.tensor([0.0, 0.0, 1.0], device=DEV, dtype=torch.float64)
        at = torch.tensor([pan[0] - vel[0], pan[1] - vel[1]], device=DEV, dtype=torch.float64)
        bg = torch.tensor(pan, device=DEV, dtype=torch.float64)
        f = {"radiance": _noisy(clean, g), "normal": torch.where(disk, up, normal), "wpos": torch.where(disk, on, wpos),
             "motion": torch.where(disk, at, bg).expand(h, w, 2), "clean": clean}
        out.append({k: v.float().contiguous() for k, v in f.items()})
    prev, cur = out
    length = torch.randint(1, 6, (h, w), device=DEV, generator=g).float()
    prev = {"radiance": (prev["clean"] + prev["radiance"]) * 0.5, "length": length, "normal": prev["normal"],
            "wpos": prev["wpos"]}
    return cur, prev


def _mr_inputs(case, seed):
    h, w, levels = case["h"], case["w"], case["levels"]
    g, m = _gen(seed), len(_kernels(case))
    f = _frame(1000 * seed, h, w)
    mod = f["albedo"] + EPS_ALBEDO
    heads = [_head(g, 1, h >> l, w >> l, m) for l in range(levels)]
    alphas = [torch.rand((h >> l, w >> l), device=DEV, generator=g) for l in range(levels - 1)]
    return heads, f["radiance"] / mod, alphas, mod


# ---------------------------------------------------------------- the calls
def prepare(case, seed):
    kind = case["kind"]
    if kind in ("denoise", "batch", "train"):
        frames, cfg, blob = _frames(case, seed), _config(case["net"]), _weights(case["net"], seed)
        scales = None
        if case["prec"] == "fp8":
            # calibrated once on a small frame and kept with two digits, as a program would store them
            s = wskp.calibrate_fp8_scales(cfg, blob, _frame(seed + 5, 256, 256))
            scales = np.array([float("%.1e" % v) for v in s], np.float32)
        dn = wskp.Denoiser(cfg, blob, case["prec"], act_scales=scales)
        hs, ws = zip(*_sizes(case))
        if kind != "denoise":
            for f in frames:
                f["out"] = torch.empty_like(f["radiance"])
        st = {"kind": kind, "dn": dn, "frames": frames}
        if kind == "train":
            st["targets"] = [f["clean"] for f in frames]
            st["ws"] = torch.empty(wskp.wskp_train_workspace_size(dn.h, hs, ws), dtype=torch.uint8, device=DEV)
            st["m"], st["v"] = _moments(case["net"], seed)
            st["grad"], st["weights"] = torch.empty_like(st["m"]), torch.empty_like(st["m"])
            st["loss"] = torch.empty(1, dtype=torch.float32, device=DEV)
        else:
            dn.workspace(list(hs), list(ws))
        return st
    if kind in ("decode", "decode_grad"):
        head, c, mod, g = _decode_inputs(case, seed)
        st = {"kind": kind, "dn": _decode_handle(_kernels(case)), "head": head, "c": c, "mod": mod, "g": g}
        if kind == "decode":
            st["out"] = torch.empty_like(c)
        else:
            head.requires_grad_(True)
            c.requires_grad_(True)
        return st
    if kind == "temporal":
        cur, prev = _temporal_inputs(case, seed)
        return {"kind": kind, "dn": _decode_handle((3,)), "cur": cur, "prev": prev,
                "out": torch.empty_like(cur["radiance"]), "length": torch.empty_like(prev["length"])}
    heads, c, alphas, mod = _mr_inputs(case, seed)
    dn = _decode_handle(_kernels(case))
    need = wskp.wskp_mr_workspace_size(dn.h, case["levels"], case["h"], case["w"])
    return {"kind": kind, "dn": dn, "heads": heads, "c": c, "alphas": alphas, "mod": mod,
            "ws": torch.empty(need, dtype=torch.uint8, device=DEV)}


def run(state):
    kind, dn = state["kind"], state["dn"]
    if kind == "denoise":
        return dn(state["frames"][0])
    if kind == "batch":
        dn.batch(state["frames"])
        return [f["out"] for f in state["frames"]]
    if kind == "train":
        wskp.wskp_train_grads(dn.h, state["frames"], state["targets"], state["grad"], state["loss"], state["ws"], EPS_SMAPE)
        # the weights, not the gradient, come back: a change of rounding anywhere in the forward pass carries a few
        # pre-activations across the ReLU's zero, which moves the raw gradient by up to 6e-5 of its norm
        wskp.wskp_adam(dn.h, state["grad"], state["m"], state["v"], STEP, LR, BETA1, BETA2, ADAM_EPS)
        wskp.wskp_get_weights(dn.h, state["weights"])
        return {"weights": state["weights"], "m": state["m"], "v": state["v"], "loss": state["loss"],
                "out": [f["out"] for f in state["frames"]]}
    if kind == "decode":
        wskp.wskp_decode(dn.h, state["head"], state["c"], state["mod"], state["out"])
        return state["out"]
    if kind == "decode_grad":
        y = wskp.WskpDecode.apply(dn.h, state["head"], state["c"], state["mod"])
        gh, gc = torch.autograd.grad(y, (state["head"], state["c"]), state["g"])
        return {"y": y, "grad_head": gh, "grad_c": gc}
    if kind == "temporal":
        cur = state["cur"]
        wskp.wskp_temporal(dn.h, cur["radiance"], cur["normal"], cur["wpos"], cur["motion"], state["prev"],
                           state["out"], state["length"])
        return state["out"], state["length"]
    return wskp.mr_reconstruct(dn.h, state["heads"], state["c"], state["alphas"], state["mod"], ws=state["ws"])


def work(case):
    kind = case["kind"]
    if kind in ("denoise", "batch", "train"):
        dims, k = _convs(case["net"])
        levels, _, kernels, _, _ = NETS[case["net"]]
        lev = list(range(levels)) + list(range(levels - 2, -1, -1)) + [0]
        px = sum(h * w for h, w in _sizes(case))
        conv = sum(2.0 * k * k * ci * co * px / 4 ** l for (ci, co), l in zip(dims, lev))
        wbytes = 4.0 * sum(co * ci * k * k + co for ci, co in dims)
        dec = 30.0 * len(kernels) * px
        if kind == "train":
            # forward, weight gradients, and input gradients of all but the first conv; reads the frames and
            # the targets, writes the outputs; reads and writes the weights and the moments
            first = 2.0 * k * k * dims[0][0] * dims[0][1] * px
            return {"bytes": px * (40 + 12 + 12) + 6 * wbytes, "flops": 3 * conv - first + 3 * dec}
        return {"bytes": px * (40 + 12) + wbytes * {"fp32": 1, "bf16": 0.5, "fp8": 0.25}[case["prec"]], "flops": conv + dec}
    if kind in ("decode", "decode_grad"):
        px, m = case["n"] * case["h"] * case["w"], len(_kernels(case))
        if kind == "decode":
            return {"bytes": px * (8.0 * m + 36), "flops": 30.0 * m * px}
        # forward (head, c, mod in; y out), backward (head, c, mod, g in; grad_head, grad_c out)
        return {"bytes": px * (8.0 * m + 36 + 16.0 * m + 48), "flops": 100.0 * m * px}
    if kind == "temporal":
        px = case["h"] * case["w"]
        return {"bytes": px * 100.0, "flops": px * 150.0}
    px = sum((case["h"] >> l) * (case["w"] >> l) for l in range(case["levels"]))
    m = len(_kernels(case))
    return {"bytes": px * (8.0 * m + 4) + case["h"] * case["w"] * 36.0, "flops": 30.0 * m * px + 20.0 * px}


# ---------------------------------------------------------------- float64 evaluation
def _conv(x, w, b):
    """x [H,W,Ci] or [N,H,W,Ci], w [Co,Ci,k,k]: zero-padded cross-correlation."""
    k = w.shape[-1]
    r = k // 2
    h, wd = x.shape[-3], x.shape[-2]
    xp = F.pad(x, (0, 0, r, r, r, r))
    y = b
    for dy in range(k):
        for dx in range(k):
            y = y + xp[..., dy:dy + h, dx:dx + wd, :] @ w[:, :, dy, dx].t()
    return y


def _pool(x):
    return 0.25 * (x[..., 0::2, 0::2, :] + x[..., 0::2, 1::2, :] + x[..., 1::2, 0::2, :] + x[..., 1::2, 1::2, :])


def _up(x):
    return x.repeat_interleave(2, -3).repeat_interleave(2, -2)


def _box(x, k):
    """k x k window sums over [..., H, W, C], windows truncated at the border."""
    r = k // 2
    h, w = x.shape[-3], x.shape[-2]
    xp = F.pad(x, (0, 0, 0, 0, r, r))
    x = sum(xp[..., d:d + h, :, :] for d in range(k))
    xp = F.pad(x, (0, 0, r, r))
    return sum(xp[..., d:d + w, :] for d in range(k))


def _decode64(weights, logits, c, kernels, floor=None):
    """Filtered and blended c (no remodulation); ``floor``: per-map divisor floors (default EPS_NORM)."""
    alpha = torch.softmax(logits, -1)
    y = 0.0
    for i, k in enumerate(kernels):
        wi = weights[..., i:i + 1]
        s = _box(wi, k).clamp_min(EPS_NORM if floor is None else floor[i])
        y = y + alpha[..., i:i + 1] * (_box(wi * c, k) / s)
    return y


def _net64(case, params, f):
    """The denoised frame(s) from preprocessed float64 buffers."""
    levels, _, kernels, act, _ = NETS[case["net"]]
    r, a, n, d = f
    x = torch.cat([r.clamp(0, 1) ** (1.0 / GAMMA), a, (n + 1) * 0.5, ((d - NEAR) / (FAR - NEAR)).clamp(0, 1)], -1)
    e = []
    for l in range(levels):
        e.append(torch.relu(_conv(x if l == 0 else _pool(e[-1]), *params[l])))
    u = e[-1]
    for i, l in enumerate(range(levels - 2, -1, -1)):
        u = torch.relu(_conv(torch.cat([_up(u), e[l]], -1), *params[levels + i]))
    h = _conv(u, *params[-1])
    m = len(kernels)
    mod = a + EPS_ALBEDO
    if act == "exp":
        # a common factor of a map's weights leaves the ratios alone
        top = [h[..., i].max() for i in range(m)]
        w = torch.stack([(h[..., i] - top[i]).exp() for i in range(m)], -1)
        floor = [EPS_NORM * float((-t).exp()) for t in top]
    else:
        w, floor = F.softplus(h[..., :m], threshold=700), None
    return _decode64(w, h[..., m:], r / mod, kernels, floor) * mod


def _params64(case, seed):
    dims, k = _convs(case["net"])
    blob, out, o = torch.from_numpy(_weights(case["net"], seed)).to(DEV).double(), [], 0
    for ci, co in dims:
        n = co * ci * k * k
        out.append((blob[o:o + n].view(co, ci, k, k), blob[o + n:o + n + co]))
        o += n + co
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("denoise", "batch", "train"):
        params = _params64(case, seed)
        frames = [{k: v.double() for k, v in f.items()} for f in _frames(case, seed)]
        buf = lambda f: (f["radiance"], f["albedo"], f["normal"], f["depth"])  # noqa: E731
        if kind != "train":
            out = [_net64(case, params, buf(f)) for f in frames]
            return out[0] if kind == "denoise" else out
        flat = [p.clone().requires_grad_(True) for wb in params for p in wb]
        params = list(zip(flat[0::2], flat[1::2]))
        total = sum(f["clean"].numel() for f in frames)
        outs, loss, grads = [], 0.0, [torch.zeros_like(p) for p in flat]
        for f in frames:
            y = _net64(case, params, buf(f))
            part = ((y - f["clean"]).abs() / (y.abs() + f["clean"].abs() + EPS_SMAPE)).sum() / total
            for acc, g in zip(grads, torch.autograd.grad(part, flat)):
                acc += g
            outs.append(y.detach())
            loss = loss + part.detach()
        grad, w = torch.cat([g.reshape(-1) for g in grads]), torch.cat([p.detach().reshape(-1) for p in flat])
        m, v = (t.double() for t in _moments(case["net"], seed))
        m = BETA1 * m + (1 - BETA1) * grad
        v = BETA2 * v + (1 - BETA2) * grad * grad
        w = w - LR * (m / (1 - BETA1 ** STEP)) / ((v / (1 - BETA2 ** STEP)).sqrt() + ADAM_EPS)
        return {"weights": w, "m": m, "v": v, "loss": loss.reshape(1), "out": outs}
    if kind in ("decode", "decode_grad"):
        ks = _kernels(case)
        head, c, mod, g = (t.double() for t in _decode_inputs(case, seed))
        m = len(ks)
        if kind == "decode":
            return _decode64(head[..., :m], head[..., m:], c, ks) * mod
        head.requires_grad_(True)
        c.requires_grad_(True)
        y = _decode64(head[..., :m], head[..., m:], c, ks) * mod
        gh, gc = torch.autograd.grad(y, (head, c), g)
        return {"y": y.detach(), "grad_head": gh, "grad_c": gc}
    if kind == "temporal":
        return _temporal64(*_temporal_inputs(case, seed))
    heads, c, alphas, mod = _mr_inputs(case, seed)
    ks, levels = _kernels(case), case["levels"]
    m, cs, fs = len(ks), [c.double()], []
    for l in range(1, levels):
        cs.append(_pool(cs[-1]))
    for l in range(levels):
        h = heads[l][0].double()
        fs.append(_decode64(h[..., :m], h[..., m:], cs[l], ks))
    o = fs[-1]
    for l in range(levels - 2, -1, -1):
        al = alphas[l].double()[..., None]
        o = fs[l] - al * _up(_pool(fs[l])) + al * _up(o)
    return o * mod.double()


def _temporal64(cur, prev):
    h, w, _ = cur["radiance"].shape
    r, n, wp, mv = (cur[k].double() for k in ("radiance", "normal", "wpos", "motion"))
    x, y = _grid(h, w)
    qx, qy = x - 0.5 + mv[..., 0], y - 0.5 + mv[..., 1]
    x0, y0 = qx.floor(), qy.floor()
    fx, fy = qx - x0, qy - y0
    tol2, ntol = float(np.float32(0.02)) ** 2, float(np.float32(0.9))
    s = torch.zeros_like(fx)
    ls, hs = torch.zeros_like(fx), torch.zeros_like(r)
    for t in range(4):
        tx, ty = (x0 + (t & 1)).long(), (y0 + (t >> 1)).long()
        ok = (tx >= 0) & (tx < w) & (ty >= 0) & (ty < h)
        q = torch.where(ok, ty * w + tx, 0)
        take = lambda k, c: prev[k].double().reshape(h * w, c)[q.reshape(-1)].reshape(h, w, c)  # noqa: E731
        ok &= ((take("wpos", 3) - wp) ** 2).sum(-1) <= tol2
        ok &= (take("normal", 3) * n).sum(-1) >= ntol
        wt = torch.where(ok, (fx if t & 1 else 1 - fx) * (fy if t >> 1 else 1 - fy), 0.0)
        s += wt
        ls += wt * take("length", 1)[..., 0]
        hs += wt[..., None] * take("radiance", 3)
    has = s > 0
    d = torch.where(has, s, 1.0)
    length = ls / d
    al = (1.0 / (length + 1.0)).clamp_min(float(np.float32(0.2)))[..., None]
    out = torch.where(has[..., None], (1 - al) * (hs / d[..., None]) + al * r, r)
    return out, torch.where(has, length + 1.0, 1.0)
