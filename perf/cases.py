"""The work that programs built on this package have it do, as timed cases.

Every case is one pass through public entry points: the fitting loop of one
frame (plain, quantisation-aware, or restricted to a P-frame's changed
Gaussians), the batched loop, the differentiable render, the initialisers,
the learned initialiser's training step and its use on a P-frame, and
quantisation.  Sizes are those of `workloads.py`, `bench.py` and the tests:
from a 96x64 crop to 1920x1080 frames with up to 50,000 Gaussians.

`exact` computes the same outputs in 64 bits with plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2505_09324_amd import _lib, autograd, synth

DEV = "cuda"
LR = (2e-2, 5e-3, 5e-3)     # mean, Cholesky vector, colour
COLD, ONGOING = "cold", "ongoing"
ONGOING_STEP = 200          # Adam steps an ongoing fit has behind it
SP_ROUNDS = 10              # superpixel rounds
SP_COMPACT = 0.1
CNN_LR = 1e-3
# in-cutoff pixels per frame pixel of the content-aware initialisation: a
# Gaussian's cutoff ellipse covers 9 pi l1 l3 with l = sqrt(1 / (n pmf)) / 2
PAIRS_PER_PIXEL = 9.0 * math.pi / 4.0


# ------------------------------------------------------------------- cases --
def listed():
    return [
        # one stretch of encoding a 1080p frame: the package's headline use
        dict(name="fit-1080p", kind="fit", W=1920, H=1080, N=30000, tile=32, ppl=2, iters=20,
             adam=ONGOING, bits=0),
        # the paper's Table 1 setting from its initialisation: launch bound
        dict(name="fit-360p", kind="fit", W=640, H=360, N=1000, tile=32, ppl=2, iters=50,
             adam=COLD, bits=0),
        # quantisation-aware encoding (Sec. 3.3.A)
        dict(name="fit-720p-qat", kind="fit", W=1280, H=720, N=15000, tile=32, ppl=2, iters=20,
             adam=ONGOING, bits=6),
        # a P-frame of a call: pick the Gaussians under changed pixels, refit
        # only those, with a PSNR check every 10 iterations
        dict(name="pframe-1080p", kind="pframe", W=1920, H=1080, N=30000, tile=32, ppl=2,
             iters=20, tau=0.02),
        # independent frames of mixed sizes fitted in lockstep
        dict(name="batch-12", kind="batch", tile=32, ppl=2, iters=10,
             sizes="1920x1080 320x240 1280x720 640x480 320x240 1920x1080 640x480 1280x720 "
                   "1920x1080 640x480 320x240 1280x720"),
        # the differentiable render under a torch loss: a whole frame, and a
        # ragged crop where the calls themselves count
        dict(name="autograd-1080p", kind="autograd", W=1920, H=1080, N=30000, tile=16),
        dict(name="autograd-crop", kind="autograd", W=123, H=90, N=300, tile=16),
        # initialising a frame: content-aware draws, then superpixels
        dict(name="init-1080p", kind="init", W=1920, H=1080, N=30000),
        dict(name="init-360p", kind="init", W=640, H=360, N=1000),
        # the learned initialiser: one training step, and re-initialising the
        # changed tiles of a warm-started P-frame
        dict(name="train-1080p", kind="train", W=1920, H=1080, N=30000),
        dict(name="reinit-1080p", kind="predict", W=1920, H=1080, N=30000, pframe=True, tau=0.001),
        # post-training quantisation of a fitted frame and its bit count
        dict(name="ptq-30k", kind="ptq", N=30000, bits_chol=6, bits_rgb=6),
    ]


def _loguniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _frame_size(rng, lo=96 * 64, hi=1920 * 1080):
    area, aspect = _loguniform(rng, lo, hi), rng.uniform(4 / 3, 16 / 9)
    w = min(1920, max(16, round(math.sqrt(area * aspect))))
    return w, min(1080, max(16, round(area / w)))


def draw(rng):
    kind = rng.choice(["fit", "fit", "pframe", "batch", "autograd", "autograd", "init", "train",
                       "predict", "ptq"])
    if kind == "ptq":
        return dict(kind=kind, N=round(_loguniform(rng, 1000, 50000)),
                    bits_chol=rng.randint(4, 10), bits_rgb=rng.randint(4, 10))
    if kind == "batch":
        dims = rng.choices(synth.BATCH_SIZES, k=rng.randint(3, 9))
        return dict(kind=kind, tile=rng.choice([16, 32]), ppl=rng.choice([1, 2]),
                    iters=rng.randint(3, 10), sizes=" ".join(f"{w}x{h}" for w, h in dims))
    W, H = _frame_size(rng)
    # pixels per Gaussian: 41 (the batched workload's 1080p) to 230 (Table 1)
    N = max(32, min(50000, round(W * H / _loguniform(rng, 41, 230))))
    if kind == "fit":
        bits = rng.choice([0, 0, 6, 8])
        return dict(kind=kind, W=W, H=H, N=N, tile=rng.choice([16, 32]), ppl=rng.choice([1, 2]),
                    iters=rng.randint(5, 30), adam=ONGOING, bits=bits)
    if kind == "pframe":
        return dict(kind=kind, W=W, H=H, N=N, tile=32, ppl=2, iters=10 * rng.randint(1, 2),
                    tau=rng.choice([0.02, 0.05]))
    if kind == "autograd":
        return dict(kind=kind, W=W, H=H, N=N, tile=rng.choice([16, 16, 32]))
    if kind == "predict":
        return dict(kind=kind, W=W, H=H, N=N, pframe=rng.random() < 0.5,
                    tau=rng.choice([0.001, 0.01]))
    return dict(kind=kind, W=W, H=H, N=N)


# ------------------------------------------------------------------ inputs --
def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _draws(N, seed):
    """Device tensors of the content-aware initialiser's random draws."""
    d = synth.init_draws(N, seed)
    return [_t(a) for a in (d.pick_roi, d.jit_roi, d.pick_out, d.jit_out)]


def _content_init(frame, mask, N, seed):
    return [p.contiguous() for p in _lib.init_plain(frame, mask.to(torch.uint8), *_draws(N, seed))]


def _adam_state(N, W, H, adam):
    """m, v, step: zeros at a cold start; an ongoing fit's second moments are
    of the order of its gradients, which scale with 1 / (3 H W)."""
    m, v = torch.zeros(8 * N, device=DEV), torch.zeros(8 * N, device=DEV)
    step = torch.zeros(1, dtype=torch.int32, device=DEV)
    if adam == ONGOING:
        v.fill_((0.5 / (3.0 * W * H)) ** 2)
        step.fill_(ONGOING_STEP)
    return [m, v, step]


def _sizes(case):
    dims = [tuple(int(x) for x in s.split("x")) for s in case["sizes"].split()]
    return [(w, h, synth.batch_gaussian_count(w, h)) for w, h in dims]


def _fitted(N, seed):
    """Gaussians with the spread of a fitted 1080p frame."""
    rng = np.random.Generator(np.random.PCG64(seed))
    xy = rng.uniform(0.0, 1.0, (N, 2)) * (1920.0, 1080.0)
    l1, l3 = np.exp(rng.normal(0.8, 0.5, (2, N)))
    chol = np.stack([l1, rng.normal(0.0, 0.6, N), l3], 1)
    rgb = rng.normal(0.12, 0.09, (N, 3))
    return [_t(a.astype(np.float32)) for a in (xy, chol, rgb)]


def prepare(case, seed):
    """What a program holds before the call: frames and Gaussians on the
    GPU, workspaces, the network and prepared calls."""
    kind, s = case["kind"], {"case": case}
    if kind == "ptq":
        s["theta"] = _fitted(case["N"], seed)
        return s
    if kind == "batch":
        return _prepare_batch(case, seed, s)
    W, H, N = case["W"], case["H"], case["N"]
    if kind == "pframe":      # only the subject's mouth moves between frames
        prev, mask = synth.make_talking_frame_torch(W, H, seed, seed % 9, DEV)
        s["frame"] = synth.make_talking_frame_torch(W, H, seed, seed % 9 + 1, DEV)[0]
    else:
        t = seed % 60 + 1
        prev, _ = synth.make_frame_torch(W, H, seed, t - 1, DEV)
        s["frame"], mask = synth.make_frame_torch(W, H, seed, t, DEV)
    s["prev"] = prev
    if kind == "init":
        s["mask"] = mask.to(torch.uint8).contiguous()
        s["draws"] = _draws(N, seed + 1)
        s["picked"] = torch.empty(N, dtype=torch.int32, device=DEV)
        return s
    s["theta"] = _content_init(prev, mask, N, seed + 1)
    if kind == "autograd":
        s["theta"] = [p.requires_grad_() for p in s["theta"]]
        s["grad"] = (s["frame"] - 0.5) * (2.0 / (3.0 * H * W))
    elif kind in ("train", "predict"):
        s["net"] = _lib.CNNInit(H, W, seed=seed + 2, device=DEV)
        s["net"].step_count.fill_(ONGOING_STEP)
        s["net"].v.fill_(1e-6)
        s["master0"] = s["net"].master.clone()
        s["head"] = torch.empty(73, s["net"].TY, s["net"].TX, device=DEV)
        s["work"] = [p.clone() for p in s["theta"]]
        s["stats"] = torch.zeros(4, dtype=torch.int32, device=DEV)
    else:                     # one-frame fits
        shape = _lib.make_shape(W, H, N, case["tile"], px_per_lane=case["ppl"])
        s["start"] = s["theta"] + _adam_state(N, W, H, case.get("adam", COLD))
        s["work"] = [p.clone() for p in s["start"]]
        s["trace"] = torch.zeros(ONGOING_STEP + case["iters"] + 8, device=DEV)
        s["shape"], s["ws"] = shape, _lib.alloc_workspace(shape, DEV)
        s["active"] = torch.zeros(N, dtype=torch.uint8, device=DEV)
        s["counts"] = torch.zeros(2, dtype=torch.int32, device=DEV)
        pf = kind == "pframe"
        opts = _lib.fit_opts(case["iters"], 10 if pf else 50, 60.0 if pf else 0.0,
                             cfg=_lib.adam_cfg(LR), active=s["active"] if pf else None,
                             qat=(case["bits"],) * 2 if case.get("bits") else None)
        s["fit"] = _lib.FitCall(shape, s["frame"], *s["work"], s["trace"], s["ws"], opts)
    return s


def _prepare_batch(case, seed, s):
    sizes = s["sizes"] = _sizes(case)
    frames, theta = [], []
    for i, (w, h, n) in enumerate(sizes):
        f, mask = synth.make_frame_torch(w, h, seed + i, seed % 60, DEV)
        frames.append(f.reshape(-1))
        theta.append(_content_init(f, mask, n, seed + 1000 + i))
    Nt = sum(n for _, _, n in sizes)
    m, v, step = _adam_state(Nt, 1, 1, COLD)
    for lo, d in ((0, 2), (2 * Nt, 3), (5 * Nt, 3)):
        k = lo
        for w, h, n in sizes:
            v[k:k + d * n] = (0.5 / (3.0 * w * h)) ** 2
            k += d * n
    step.fill_(ONGOING_STEP)
    s["targets"] = torch.cat(frames)
    s["start"] = [torch.cat(p).contiguous() for p in zip(*theta)] + [m, v, step]
    s["work"] = [p.clone() for p in s["start"]]
    s["trace"] = torch.zeros(ONGOING_STEP + case["iters"] + 8, len(sizes), device=DEV)
    s["ws"] = torch.empty(_lib.batch_workspace_bytes(sizes, case["tile"], case["ppl"]),
                          dtype=torch.uint8, device=DEV)
    s["opts"] = _lib.fit_opts(case["iters"], 50, cfg=_lib.adam_cfg(LR))
    return s


# -------------------------------------------------------------------- pass --
def _restart(s):
    """The frame's starting Gaussians and optimiser state into the buffers
    that the fit updates in place."""
    for a, b in zip(s["work"], s["start"]):
        a.copy_(b)


def run(s):
    case = s["case"]
    return {"fit": _run_fit, "pframe": _run_pframe, "batch": _run_batch,
            "autograd": _run_autograd, "init": _run_init, "train": _run_train,
            "predict": _run_predict, "ptq": _run_ptq}[case["kind"]](s, case)


def _fit_outputs(s):
    return dict(zip(("xy", "chol", "rgb", "m", "v", "step"), s["work"]), trace=s["trace"])


def _run_fit(s, case):
    _restart(s)
    s["fit"]()
    return _fit_outputs(s)


def _run_pframe(s, case):
    _restart(s)
    xy, chol = s["work"][:2]
    _lib.project_bin(s["shape"], xy, chol, s["ws"])
    _lib.select_changed(s["shape"], s["ws"], xy, chol, s["frame"], s["prev"], case["tau"],
                        active=s["active"], counts=s["counts"])
    s["fit"]()
    return dict(_fit_outputs(s), active=s["active"], counts=s["counts"])


def _run_batch(s, case):
    _restart(s)
    _lib.fit_batch(s["sizes"], case["tile"], case["ppl"], s["targets"], *s["work"], s["trace"],
                   s["ws"], s["opts"])
    return _fit_outputs(s)


def _run_autograd(s, case):
    img = autograd.render(*s["theta"], case["W"], case["H"], case["tile"])
    grads = torch.autograd.grad(img, s["theta"], s["grad"])
    return {"img": img.detach(), "g_xy": grads[0], "g_chol": grads[1], "g_rgb": grads[2]}


def _run_init(s, case):
    xy, chol, rgb = _lib.init_plain(s["frame"], s["mask"], *s["draws"], picked=s["picked"])
    k = s["draws"][0].shape[0]
    _lib.init_superpixel(s["frame"], s["mask"], s["picked"][:k], xy[:k], chol[:k], rgb[:k],
                         iters=SP_ROUNDS, compactness=SP_COMPACT)
    return {"xy": xy, "chol": chol, "rgb": rgb, "picked": s["picked"]}


def _run_train(s, case):
    net = s["net"]
    net.forward(s["frame"], s["prev"])
    net.set_targets(*s["theta"])
    loss = net.backward()
    net.step(lr=CNN_LR)
    return {"loss": loss, "master": net.master, "m": net.m, "v": net.v, "step": net.step_count}


def _run_predict(s, case):
    net = s["net"]
    if not case["pframe"]:    # an I-frame: every Gaussian from the network
        net.forward(s["frame"], None, head_out=s["head"])
        xy, chol, rgb, n = net.decode(case["N"], *s["theta"])
        return {"head": s["head"], "xy": xy, "chol": chol, "rgb": rgb, "n": n}
    for a, b in zip(s["work"], s["theta"]):
        a.copy_(b)
    net.forward(s["frame"], s["prev"], head_out=s["head"])
    net.pframe_replace(s["frame"], s["prev"], case["tau"], *s["work"], stats=s["stats"])
    return dict(zip(("xy", "chol", "rgb"), s["work"]), head=s["head"], stats=s["stats"])


def _run_ptq(s, case):
    return _lib.ptq(*s["theta"], case["bits_chol"], case["bits_rgb"])


# -------------------------------------------------------------------- work --
def _conv_macs(W, H):
    out, h, w, cin, act = 0.0, H, W, 6, 0.0
    for i in range(5):
        if i < 4:
            h, w = (h + 1) // 2, (w + 1) // 2
        cout = 64 if i < 4 else 73
        out += float(h * w * cout * 9 * cin)
        act += float(h * w * cout)
        cin = cout
    return out, act


def work(case):
    """Per pass: a fit reads its target and reads and writes parameters and
    moments every iteration, with 16 forward and 36 backward operations per
    in-cutoff (pixel, Gaussian) pair; a superpixel round scores about nine
    centres per ROI pixel; the network's passes are its convolutions and its
    16-bit activations written and read once per direction."""
    kind = case["kind"]
    if kind == "ptq":
        return {"bytes": 64.0 * case["N"], "flops": 40.0 * case["N"]}
    if kind == "batch":
        px = sum(w * h for w, h, _ in _sizes(case))
        n = sum(n for _, _, n in _sizes(case))
        return {"bytes": case["iters"] * (12.0 * px + 192.0 * n),
                "flops": case["iters"] * 52.0 * PAIRS_PER_PIXEL * px}
    px, n = float(case["W"] * case["H"]), float(case["N"])
    if kind == "fit":
        return {"bytes": case["iters"] * (12.0 * px + 192.0 * n),
                "flops": case["iters"] * 52.0 * PAIRS_PER_PIXEL * px}
    if kind == "pframe":      # the backward covers the few selected Gaussians
        return {"bytes": 24.0 * px + case["iters"] * (12.0 * px + 32.0 * n),
                "flops": case["iters"] * 17.0 * PAIRS_PER_PIXEL * px}
    if kind == "autograd":
        return {"bytes": 24.0 * px + 64.0 * n, "flops": 52.0 * PAIRS_PER_PIXEL * px}
    if kind == "init":
        return {"bytes": 13.0 * px + 64.0 * n + SP_ROUNDS * 0.25 * 12.0 * px,
                "flops": SP_ROUNDS * 0.25 * px * 9 * 11.0}
    macs, act = _conv_macs(case["W"], case["H"])
    if kind == "train":
        return {"bytes": 24.0 * px + 12.0 * act + 32.0 * n, "flops": 6.0 * macs}
    return {"bytes": 24.0 * px + 4.0 * act + 64.0 * n, "flops": 2.0 * macs}


# ------------------------------------------------------------------- exact --
def _pairs(xy, chol, W, H):
    """Every (Gaussian, pixel) inside the 3-sigma cutoff: Gaussian, pixel,
    whitened offsets and weight."""
    mx, my = xy.unbind(1)
    l1, l2, l3 = chol.unbind(1)
    rx, ry = 3 * l1.abs(), 3 * torch.sqrt(l2 * l2 + l3 * l3)
    x0 = torch.ceil(mx - rx - 0.5).clamp(min=0).long()
    y0 = torch.ceil(my - ry - 0.5).clamp(min=0).long()
    nx = (torch.floor(mx + rx - 0.5).clamp(max=W - 1).long() - x0 + 1).clamp(min=0)
    ny = (torch.floor(my + ry - 0.5).clamp(max=H - 1).long() - y0 + 1).clamp(min=0)
    cnt = nx * ny
    n = torch.repeat_interleave(torch.arange(len(cnt), device=DEV), cnt)
    k = torch.arange(len(n), device=DEV) - (cnt.cumsum(0) - cnt)[n]
    x, y = x0[n] + k % nx[n], y0[n] + k // nx[n]
    u1 = (x + 0.5 - mx[n]) / l1[n]
    u2 = (y + 0.5 - my[n] - l2[n] * u1) / l3[n]
    q = u1 * u1 + u2 * u2
    keep = q <= 9
    return n[keep], (y * W + x)[keep], u1[keep], u2[keep], torch.exp(-0.5 * q[keep])


def _render(theta, W, H, pairs):
    n, p, _, _, w = pairs
    return torch.zeros(3, H * W, dtype=torch.float64, device=DEV).index_add_(
        1, p, w * theta[2].T[:, n])


def _gradients(theta, g, pairs):
    """dL/d(mean, Cholesky vector, colour) for dL/dC = g [3, HW]."""
    n, p, u1, u2, w = pairs
    _, chol, rgb = theta
    gp = g[:, p]
    s = (gp * rgb.T[:, n]).sum(0) * w
    v2 = u2 / chol[n, 2]
    v1 = (u1 - chol[n, 1] * v2) / chol[n, 0]
    rows = torch.stack([s * v1, s * v2, s * v1 * u1, s * v2 * u1, s * v2 * u2, *(gp * w)])
    out = torch.zeros(8, len(rgb), dtype=torch.float64, device=DEV).index_add_(1, n, rows)
    return out[:2].T, out[2:5].T, out[5:].T


def _fit64(start, target, iters, W, H, active=None):
    """The fitting loop in 64 bits: (theta, m, v, losses)."""
    theta = [p.double() for p in start[:3]]
    m, v, step = start[3].double(), start[4].double(), int(start[5])
    f32 = lambda x: float(np.float32(x))                               # noqa: E731
    b1, b2, eps = f32(0.9), f32(0.999), f32(1e-8)
    N = len(theta[0])
    lr = torch.cat([torch.full((d * N,), f32(x), dtype=torch.float64, device=DEV)
                    for d, x in zip((2, 3, 3), LR)])
    if active is not None:
        on = torch.cat([active.bool()[:, None].expand(N, d).reshape(-1) for d in (2, 3, 3)])
    T = target.double().reshape(3, -1)
    losses = []
    for _ in range(iters):
        pairs = _pairs(theta[0], theta[1], W, H)
        r = _render(theta, W, H, pairs) - T
        losses.append((r * r).mean())
        g = torch.cat([x.reshape(-1) for x in _gradients(theta, r * (2 / T.numel()), pairs)])
        step += 1
        m1, v1 = b1 * m + (1 - b1) * g, b2 * v + (1 - b2) * g * g
        flat = torch.cat([p.reshape(-1) for p in theta])
        new = flat - lr * (m1 / (1 - b1 ** step)) / (torch.sqrt(v1 / (1 - b2 ** step)) + eps)
        if active is not None:
            m1, v1, new = torch.where(on, m1, m), torch.where(on, v1, v), torch.where(on, new, flat)
        m, v = m1, v1
        theta = [new[:2 * N].reshape(N, 2), new[2 * N:5 * N].reshape(N, 3),
                 new[5 * N:].reshape(N, 3)]
    return theta, m, v, torch.stack(losses)


def _selected(theta, frame, prev, tau, W, H):
    """The Gaussians with a changed pixel inside their cutoff: a decision,
    taken with the 32-bit operations that define it."""
    changed = ((frame - prev).abs() > tau).any(0).reshape(-1)
    xy, chol = theta[:2]
    wide = chol.double().clone()
    wide[:, 0] *= 1.001       # candidate pixels: a slightly larger ellipse
    wide[:, 2] *= 1.001
    n, p, _, _, _ = _pairs(xy.double(), wide, W, H)
    n, p = n[changed[p]], p[changed[p]]
    dx = (p % W).float() + 0.5 - xy[n, 0]
    dy = torch.div(p, W, rounding_mode="floor").float() + 0.5 - xy[n, 1]
    u1 = dx / chol[n, 0]
    u2 = (dy - chol[n, 1] * u1) / chol[n, 2]
    active = torch.zeros(len(xy), dtype=torch.uint8, device=DEV)
    active[n[u1 * u1 + u2 * u2 <= 9]] = 1
    return active


def _exact_fit(start, frame, case, active=None):
    theta, m, v, losses = _fit64(start, frame, case["iters"], case["W"], case["H"], active)
    step0 = int(start[5])
    trace = torch.zeros(ONGOING_STEP + case["iters"] + 8, dtype=torch.float64, device=DEV)
    trace[step0:step0 + case["iters"]] = losses
    return {"xy": theta[0], "chol": theta[1], "rgb": theta[2], "m": m, "v": v, "step": None,
            "trace": trace}


def _exact_batch(case, s):
    sizes, start = s["sizes"], s["start"]
    Nt, F = sum(n for _, _, n in sizes), len(sizes)
    outs, o, px = [], 0, 0
    trace = torch.zeros(ONGOING_STEP + case["iters"] + 8, F, dtype=torch.float64, device=DEV)
    cut = lambda a, o, n: torch.cat([a[b + d * o:b + d * (o + n)] for b, d in  # noqa: E731
                                     ((0, 2), (2 * Nt, 3), (5 * Nt, 3))])
    for f, (w, h, n) in enumerate(sizes):
        st = [p[o:o + n] for p in start[:3]] + [cut(start[3], o, n), cut(start[4], o, n), start[5]]
        theta, m, v, losses = _fit64(st, s["targets"][px:px + 3 * w * h], case["iters"], w, h)
        trace[ONGOING_STEP:ONGOING_STEP + case["iters"], f] = losses
        outs.append((*theta, m, v, n))
        o, px = o + n, px + 3 * w * h
    whole = {k: torch.cat([x[i] for x in outs]) for i, k in enumerate(("xy", "chol", "rgb"))}
    for i, k in ((3, "m"), (4, "v")):
        whole[k] = torch.cat([x[i][b * x[5]:(b + d) * x[5]] for b, d in ((0, 2), (2, 3), (5, 3))
                              for x in outs])
    return dict(whole, step=None, trace=trace)


def _net_head(frame, prev, master, net, leaves=None):
    """The network in 64 bits: head [73, TY, TX]; `leaves` receives each
    layer's weight matrix and bias."""
    res = torch.zeros_like(frame) if prev is None else frame - prev
    x = torch.cat([frame, res, torch.zeros_like(frame[:2])]).double()
    for i in range(5):
        d = net.layer_info(i)
        K = 9 * d["Cin"]
        M = master[d["w_off"]:d["w_off"] + d["Mpad"] * d["Kf"]].double().reshape(d["Mpad"], d["Kf"])
        M = M.clone()
        b = master[d["b_off"]:d["b_off"] + d["Mpad"]].double().clone()
        if leaves is not None:
            leaves.append((M.requires_grad_(), b.requires_grad_(), d))
        cols = torch.nn.functional.unfold(x[None], 3, padding=1, stride=d["stride"])[0]
        # unfold orders a column (channel, tap); the weights are (tap, channel)
        cols = cols.reshape(d["Cin"], 9, -1).transpose(0, 1).reshape(K, -1)
        y = M[:d["Cout"], :K] @ cols + b[:d["Cout"], None]
        x = (torch.relu(y) if d["relu"] else y).reshape(-1, d["Hout"], d["Wout"])
    return x


def _targets64(theta, TX, TY, W, H):
    """Per 16-pixel tile the (at most 8) heaviest Gaussians centred in it, by
    index: counts [tiles], vectors [tiles, 8, 8] in 64 bits."""
    xy, chol, rgb = theta
    n = len(xy)
    ok = (xy[:, 0] >= 0) & (xy[:, 1] >= 0) & (xy[:, 0] < W) & (xy[:, 1] < H)
    tile = torch.where(ok, (xy[:, 1] / 16).floor().long() * TX + (xy[:, 0] / 16).floor().long(),
                       torch.full((n,), TX * TY, device=DEV))
    c = rgb * rgb
    mass = (chol[:, 0] * chol[:, 2]).abs() * (c[:, 0] + c[:, 1] + c[:, 2])

    def ranks(order):
        t = tile[order]
        first = torch.searchsorted(t, torch.arange(TX * TY + 1, device=DEV))
        r = torch.empty(n, dtype=torch.long, device=DEV)
        r[order] = torch.arange(n, device=DEV) - first[t]
        return r

    heavy = torch.argsort(-mass, stable=True)
    keep = (ranks(heavy[torch.argsort(tile[heavy], stable=True)]) < 8) & ok
    tile = torch.where(keep, tile, torch.full_like(tile, TX * TY))
    slot = ranks(torch.argsort(tile, stable=True))
    counts = torch.bincount(tile[keep], minlength=TX * TY)
    vec = torch.zeros(TX * TY, 8, 8, dtype=torch.float64, device=DEV)
    p, l, t = xy[keep].double(), chol[keep].double(), tile[keep]
    vec[t, slot[keep]] = torch.cat([
        ((p[:, 0] - 16 * (t % TX)) / 16)[:, None], ((p[:, 1] - 16 * (t // TX)) / 16)[:, None],
        l[:, :1].abs().log(), l[:, 1:2], l[:, 2:].abs().log(), rgb[keep].double()], 1)
    return counts, vec


def _exact_train(s, case):
    net, leaves = s["net"], []
    head = _net_head(s["frame"], s["prev"], s["master0"], net, leaves)
    z = head.reshape(73, -1).T
    counts, vec = _targets64(s["theta"], net.TX, net.TY, case["W"], case["H"])
    ce = torch.nn.functional.cross_entropy(z[:, :9], counts)
    P = z[:, 9:].reshape(-1, 8, 8)
    P = torch.cat([torch.sigmoid(P[..., :2]), P[..., 2:]], -1)
    live = torch.arange(8, device=DEV)[None] < counts[:, None]
    D = ((P[:, :, None] - vec[:, None]) ** 2).sum(-1)
    far = torch.where(live[:, :, None] & live[:, None], D, torch.full_like(D, 1e300))
    near = torch.where(live, far.min(2).values + far.min(1).values, torch.zeros_like(far[:, 0]))
    cd = (near.sum(1) / counts.clamp(min=1)).sum() / (counts > 0).sum().clamp(min=1)
    loss = ce + cd
    loss.backward()
    p = s["master0"].double()
    g = torch.zeros_like(p)
    for M, b, d in leaves:
        g[d["w_off"]:d["w_off"] + M.numel()] = M.grad.reshape(-1)
        g[d["b_off"]:d["b_off"] + b.numel()] = b.grad
    t = ONGOING_STEP + 1
    m, v = 0.1 * g, 0.999 * 1e-6 + 0.001 * g * g
    p = p - CNN_LR * (m / (1 - 0.9 ** t)) / (torch.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
    return {"loss": torch.stack([loss, ce, cd]).detach(), "master": p, "m": m, "v": v,
            "step": None}


def _exact_ptq(s, case):
    xy, chol, rgb = s["theta"]
    out = {"xy": xy.half().double()}
    bits, ranges = [], []
    for name, a, b in (("chol", chol, case["bits_chol"]), ("rgb", rgb, case["bits_rgb"])):
        cols = []
        for c in range(3):
            # the codes are decisions, taken with the 32-bit operations that
            # define them
            x, L = a[:, c], torch.tensor(float(2 ** b - 1), device=DEV)
            lo, hi = x.min(), x.max()
            code = torch.round((x - lo) * (L / (hi - lo))).clamp(0, 2 ** b - 1)
            cols.append(lo.double() + code.double() * ((hi.double() - lo.double()) / (2 ** b - 1)))
            ranges.append(torch.stack([lo, hi]).double())
            k = torch.bincount(code.long())
            pr = k[k > 0].double() / len(x)
            bits.append(-(pr * torch.log2(pr)).sum() * len(x))
        out[name] = torch.stack(cols, 1)
    bits.append(sum(bits) + 32.0 * len(xy) + 6 * 64.0)
    return dict(out, ranges=torch.stack(ranges), bits=torch.stack(bits))


def exact(case, seed):
    kind = case["kind"]
    if kind == "init" or (kind == "fit" and case["bits"]):
        return None           # K-means labels and quantiser codes: decisions all along
    s = prepare(case, seed)
    if kind == "ptq":
        return _exact_ptq(s, case)
    if kind == "batch":
        return _exact_batch(case, s)
    if kind == "fit":
        return _exact_fit(s["start"], s["frame"], case)
    if kind == "pframe":
        active = _selected(s["theta"], s["frame"], s["prev"], case["tau"], case["W"], case["H"])
        return dict(_exact_fit(s["start"], s["frame"], case, active), active=None, counts=None)
    if kind == "autograd":
        theta = [p.detach().double() for p in s["theta"]]
        pairs = _pairs(theta[0], theta[1], case["W"], case["H"])
        gx, gc, gr = _gradients(theta, s["grad"].double().reshape(3, -1), pairs)
        img = _render(theta, case["W"], case["H"], pairs).reshape(3, case["H"], case["W"])
        return {"img": img, "g_xy": gx, "g_chol": gc, "g_rgb": gr}
    if kind == "train":
        return _exact_train(s, case)
    prev = s["prev"] if case["pframe"] else None
    out = {"head": _net_head(s["frame"], prev, s["master0"], s["net"]), "xy": None, "chol": None,
           "rgb": None}
    return dict(out, **({"stats": None} if case["pframe"] else {"n": None}))
