"""The work that a user of the renderer has it do, as cases that can be timed and compared.

Each case is one call, or the few calls that belong together, through the package's public entry points
(`render`, `train`, `prune`): single views and their gradients, captured multi-view batches, one fitting
step, the importance pass, the photometric loss, the optimiser step, and a pruning round with the
post-processing that follows it. Scenes are drawn on the GPU with the distributions of the repository's
own synthetic workloads (`scenes.py`): uniform or clustered positions, N(-3.5, 0.5) log scales, N(0, 1)
opacity logits, up to four lobes with sharpness log-uniform in [1, 50], soft masks, FP32 or FP16 storage
with BF16 amplitudes, cameras on a ring of radius 6.

`exact` gives the same results in 64 bits from plain torch: a compositor without tiles or lists (every
Gaussian against every pixel, in depth order) with autograd for its gradients, the loss by convolutions,
the optimiser and pruning steps by their definitions.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2509_07021_amd import _lib as L
from paper_2509_07021_amd import prune as P
from paper_2509_07021_amd import render as R
from paper_2509_07021_amd import scenes as S
from paper_2509_07021_amd import train as T

# Sizes of the sixteen-view batch (the repository's 500k workload): four resolutions in turn.
MIXED = ((640, 360), (960, 540), (1280, 720), (1920, 1080))
# Gaussian-pixel products up to which `exact` composites by brute force (a few seconds).
EXACT_PRODUCTS = 3.0e9
TORCH_DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}

_BASE = {"kind": "view", "n": 2000, "k": 3, "sh": -1, "views": 1, "w": 128, "h": 128, "mixed": False,
         "clustered": True, "masks": False, "half": False, "ragged": False, "tile": 16, "subtile": 0,
         "det": False, "backward": True}


def _case(name=None, **kw):
    c = dict(_BASE, **kw)
    return dict({"name": name}, **c) if name else c


def listed():
    return [
        # the smallest call: a preview or a unit-test scene, one view, the default launch configuration;
        # launches, the host path and the one synchronisation are what it costs
        _case("view_2k_128", n=2000, k=3, clustered=False, w=128, h=128),
        # its differentiable form, as a first experiment in a notebook runs it
        _case("grad_2k_128", kind="grad", n=2000, k=3, clustered=False, w=128, h=128),
        # one training view of a mid-sized scene through autograd, default launch configuration
        _case("grad_200k_720p", kind="grad", n=200_000, k=4, w=1280, h=720),
        # serving: one full-HD view of a masked scene in FP32, launch as the autotuner picks it
        _case("view_1m_1080p", n=1_000_000, k=4, masks=True, w=1920, h=1080, tile=32, subtile=8),
        # the benchmark's batch: eight full-HD views, FP16 storage, forward and backward in one graph
        _case("graph_1m_half_8x1080p", kind="graph", n=1_000_000, k=4, masks=True, half=True, views=8,
              w=1920, h=1080, tile=32, subtile=8),
        # evaluation renders: sixteen views of mixed resolutions, forward only, one graph
        _case("graph_500k_16views_fwd", kind="graph", n=500_000, k=4, views=16, mixed=True, w=1920, h=1080, tile=32,
              subtile=8, backward=False),
        # the spherical-harmonic colour model at an odd image size, forward and backward
        _case("grad_sh3_300k_979x546", kind="grad", n=300_000, k=0, sh=3, w=979, h=546, tile=32, subtile=8),
        # fine-tuning a post-processed scene (0 to 3 lobes a Gaussian): render, loss, backward
        _case("fit_960k_ragged_1080p", kind="fit", n=960_000, k=3, ragged=True, w=1920, h=1080, tile=32, subtile=8),
        # importance scores of a pruning round over four views, default launch configuration
        _case("importance_200k_4x720p", kind="importance", n=200_000, k=4, masks=True, views=4, w=1280, h=720),
        # the photometric loss and its gradient on one full-HD image
        _case("loss_1080p", kind="loss", n=0, k=0, w=1920, h=1080),
        # the optimiser over every plane of a masked scene
        _case("adam_1m", kind="adam", n=1_000_000, k=4, masks=True),
        # the last round of the memory-constrained optimisation (proximal step, duals, penalties) and the
        # compaction after it
        _case("prune_1m", kind="prune", n=1_000_000, k=3, masks=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["view", "view", "grad", "grad", "graph", "fit", "importance", "loss", "adam", "prune"])
    # image sizes between the smallest and full HD, odd ones among them
    h = _log(rng, 120, 1080)
    w = min(1920, max(64, int(h * rng.uniform(1.0, 1.78))))
    half = rng.random() < 0.35
    tile, subtile = rng.choice([(16, 0), (32, 8), (32, 8), (16, 8)])
    c = dict(kind=kind, w=w, h=h, k=rng.randint(1, 4), masks=rng.random() < 0.5, half=half, tile=tile, subtile=subtile,
             clustered=rng.random() < 0.8)
    if kind == "graph":
        return _case(**dict(c, n=_log(rng, 20_000, 1_000_000), views=rng.randint(2, 8), backward=rng.random() < 0.6))
    if kind in ("view", "grad"):
        n = _log(rng, 2000, 1_500_000)
        if rng.random() < 0.25:
            return _case(**dict(c, n=min(n, 800_000), k=0, sh=rng.randint(0, 3)))
        return _case(**dict(c, n=n, ragged=rng.random() < 0.25, det=kind == "grad" and rng.random() < 0.15))
    if kind == "fit":
        return _case(**dict(c, n=_log(rng, 5000, 1_000_000), ragged=rng.random() < 0.4, views=rng.choice([1, 1, 2])))
    if kind == "importance":
        return _case(**dict(c, n=_log(rng, 5000, 500_000), views=rng.randint(1, 6)))
    if kind == "loss":
        return _case(**dict(_case(), kind="loss", n=0, k=0, views=rng.randint(1, 4), w=w, h=h))
    return _case(**dict(_case(), kind=kind, n=_log(rng, 2000, 1_600_000), k=rng.randint(1, 4), masks=rng.random() < 0.6,
                        half=half))


# ------------------------------------------------------------------ inputs ----

def _dts(case):
    return ("f16", "f16", "bf16") if case["half"] else ("f32", "f32", "f32")


def _planes(case, seed):
    """(planes, lobe offsets or None, lobes) drawn on the GPU from the seed, in their storage types."""
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 13)
    n, k = case["n"], case["k"]
    nrm = lambda *s: torch.randn(*s, generator=g, device="cuda")
    uni = lambda lo, hi, *s: torch.rand(*s, generator=g, device="cuda") * (hi - lo) + lo
    if case["clustered"]:
        centre = uni(-3.0, 3.0, 32, 3)
        sigma = uni(0.05, 0.3, 32, 3)
        rot = torch.linalg.qr(nrm(32, 3, 3).cpu().double())[0].float().cuda()
        a = torch.randint(0, 32, (n,), generator=g, device="cuda")
        z = sigma[a] * nrm(n, 3)
        pos = (centre[a] + (rot[a] * z[:, None, :]).sum(2)).clamp(-3.0, 3.0).T.contiguous()
    else:
        pos = uni(-1.0, 1.0, 3, n)
    p = {"pos": pos, "logscale": nrm(3, n) * 0.5 - 3.5, "quat": torch.nn.functional.normalize(nrm(4, n), dim=0),
         "op_logit": nrm(n), "pmask_logit": nrm(n) * 1.5 + 1.0 if case["masks"] else None}
    off, nl = None, n * k
    if case["sh"] >= 0:
        m = (case["sh"] + 1) ** 2
        sh = nrm(m, 3, n) * 0.1
        sh[0] = uni(-1.0, 1.8, 3, n)
        p.update(base=None, axis=torch.zeros(0, 3, n, device="cuda"), sharp=torch.zeros(0, n, device="cuda"),
                 amp=torch.zeros(0, 3, n, device="cuda"), lmask_logit=None, sh=sh)
    else:
        if case["ragged"]:  # each lobe survives post-processing with the paper's mean of 0.96 in 3
            nl = max(1, int(0.32 * n * k))
            kept = torch.zeros(n * k, dtype=torch.int64, device="cuda")
            kept[torch.randperm(n * k, generator=g, device="cuda")[:nl]] = 1
            off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
            off[1:] = torch.cumsum(kept.view(n, k).sum(1), 0)
            off = off.to(torch.int32)
            s3, s1, d3 = (3, nl), (nl,), 0
        else:
            s3, s1, d3 = (k, 3, n), (k, n), 1
        p.update(base=uni(0.0, 1.0, 3, n), axis=torch.nn.functional.normalize(nrm(*s3), dim=d3),
                 sharp=torch.exp(uni(0.0, math.log(50.0), *s1)), amp=nrm(*s3) * 0.2,
                 lmask_logit=nrm(*s1) * 1.5 + 0.5 if case["masks"] else None, sh=None)
    if case["kind"] == "prune":
        # what the optimisation leaves: 40% of the Gaussians faint, 68% of the others' lobes flat (fixed
        # shares, so that the compacted sizes do not depend on the draw)
        faint = torch.zeros(n, dtype=torch.bool, device="cuda")
        faint[torch.randperm(n, generator=g, device="cuda")[: (2 * n) // 5]] = True
        p["op_logit"] = torch.where(faint, (nrm(n) - 9.0).clamp(max=-6.0), p["op_logit"].clamp(min=-2.0))
        if case["masks"]:
            p["pmask_logit"] = p["pmask_logit"].clamp(min=-1.0)
        turn = torch.rand(k, n, generator=g, device="cuda") + 2.0 * faint
        flat = torch.zeros(k * n, dtype=torch.bool, device="cuda")
        flat[torch.argsort(turn.view(-1))[: int(0.68 * k * (n - (2 * n) // 5))]] = True
        flat = flat.view(k, n) | (faint & (turn < 2.68))
        p["sharp"] = torch.where(flat, uni(0.0, 0.99, k, n), p["sharp"].clamp(min=1.0))
    dts = _dts(case)
    p = {q: None if t is None else t.to(TORCH_DT[R._group_dt(q, *dts)]).contiguous() for q, t in p.items()}
    return p, off, nl


def _cams(case, seed):
    nv = case["views"]
    if not case["clustered"]:
        return [S.look_at((4.0 * math.sin(2.0 * math.pi * i / nv), -4.0 * math.cos(2.0 * math.pi * i / nv), 0.0),
                          case["w"], case["h"]) for i in range(nv)]
    cams = S.ring_cameras(nv, int(seed) % 100_000, (case["w"], case["h"]))
    if case["mixed"]:
        eyes = [-np.asarray(c.R, np.float64).T @ np.asarray(c.t, np.float64) for c in cams]
        cams = [S.look_at(e, *MIXED[i % 4]) for i, e in enumerate(eyes)]
    return cams


def _pixels(case):
    if case["mixed"]:
        return sum(MIXED[i % 4][0] * MIXED[i % 4][1] for i in range(case["views"]))
    return case["views"] * case["w"] * case["h"]


def _image_pair(case, seed):
    """An image in [-0.05, 1.05] with smooth structure, and the target it is fitted to."""
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 104729 + 7)
    npix = _pixels(case)
    base = torch.rand(3 * npix, generator=g, device="cuda")
    x = (base * 1.1 - 0.05)
    y = (x + 0.15 * torch.randn(3 * npix, generator=g, device="cuda")).clamp(0.0, 1.0)
    return x, y


def _adam_inputs(case, seed):
    """Gradients and mid-training moments for every plane."""
    p, _, _ = _planes(case, seed)
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 1299709 + 3)
    out = {}
    for q, t in p.items():
        if t is not None:
            gr = torch.randn(t.shape, generator=g, device="cuda") * 1e-3
            m = torch.randn(t.shape, generator=g, device="cuda") * 3e-4
            v = (torch.rand(t.shape, generator=g, device="cuda") + 0.1) * 1e-6
            out[q] = (gr, m, v)
    return p, out


def _admm_inputs(case, p, seed):
    n, k = case["n"], case["k"]
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 15485863 + 11)
    f = lambda *s: torch.randn(*s, generator=g, device="cuda")
    return {"o": p["op_logit"].float(), "lam_o": f(n) * 0.1, "imp": torch.exp(f(n) * 2.0),
            "s": p["sharp"].float(), "lam_s": f(k, n) * 0.1, "amp": p["amp"].float(),
            "g_o": f(n) * 1e-3, "g_s": f(k, n) * 1e-3}


def _config(case):
    return R.Config(tile=case["tile"], subtile=case["subtile"], flags=L.MEGS_FLAG_DETERMINISTIC if case["det"] else 0)


def _scene(case, seed):
    p, off, nl = _planes(case, seed)
    return R.DeviceScene(p, case["k"], *_dts(case), lobe_off=off, n_lobes=nl)


def _weights(case, seed, npix):
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 32452843 + 5)
    return torch.randn(3 * npix, generator=g, device="cuda")


_STREAM = []


def _graph_stream():
    """The one stream on which a program replays its graphs."""
    if not _STREAM:
        _STREAM.append(torch.cuda.Stream())
    return _STREAM[0]


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case, "cams": _cams(case, seed)}
    if kind == "loss":
        st["x"], st["y"] = _image_pair(case, seed)
        return st
    if kind == "adam":
        p, gmv = _adam_inputs(case, seed)
        ds = R.DeviceScene(p, case["k"], *_dts(case))
        opt = T.Adam(ds)
        opt.step_count = 999
        for q, (_, m, v) in gmv.items():
            opt.m[q].copy_(m)
            opt.v[q].copy_(v)
        st.update(ds=ds, opt=opt, grads={q: t[0] for q, t in gmv.items()})
        return st
    st["ds"] = ds = _scene(case, seed)
    st["cfg"] = _config(case)
    if kind == "prune":
        st["admm"] = _admm_inputs(case, ds.planes, seed)
        return st
    if kind == "grad":
        st["w"] = R.split_images(_weights(case, seed, _pixels(case)), st["cams"])
        st["leaves"] = [(q, t.requires_grad_(True)) for q, t in ds.planes.items() if t is not None and t.numel()]
    elif kind == "fit":
        st["y"] = _image_pair(case, seed)[1]
    elif kind == "graph":
        fr = R.forward(ds, st["cams"], st["cfg"])
        st["cfg"].pair_capacity = int(fr.state.n_pairs * 1.05) + 4096
        del fr
        dl = _weights(case, seed, _pixels(case)) if case["backward"] else None
        st["graph"] = R.Graph(ds, st["cams"], st["cfg"], with_backward=case["backward"], dl_images=dl,
                              stream=_graph_stream())
    return st


# --------------------------------------------------------------------- run ----

def _given(d):
    return {q: t for q, t in d.items() if t is not None and t.numel()}


def run(st):
    kind = st["case"]["kind"]
    if kind == "view":
        return {"images": R.render(st["ds"], st["cams"], st["cfg"])}
    if kind == "grad":
        images = R.render(st["ds"], st["cams"], st["cfg"])
        grads = torch.autograd.grad(images, [t for _, t in st["leaves"]], grad_outputs=st["w"])
        return {"images": [x.detach() for x in images], "grads": dict(zip([q for q, _ in st["leaves"]], grads))}
    if kind == "graph":
        st["graph"].launch()
        out = {"images": st["graph"].views()}
        if st["case"]["backward"]:
            out["grads"] = _given(st["graph"].grads)
        return out
    if kind == "fit":
        fr = R.forward(st["ds"], st["cams"], st["cfg"])
        loss, dl = T.photometric_loss(fr.images, st["y"], st["cams"])
        return {"images": R.split_images(fr.images, st["cams"]), "loss": loss,
                "grads": _given(R.backward(st["ds"], fr, dl))}
    if kind == "importance":
        images, imp = P.importance(st["ds"], st["cams"], st["cfg"])
        return {"images": R.split_images(images, st["cams"]), "importance": imp}
    if kind == "loss":
        loss, dl = T.photometric_loss(st["x"], st["y"], st["cams"])
        return {"loss": loss, "grad": dl}
    if kind == "adam":
        st["opt"].step(st["grads"])
        return {"planes": _given(st["ds"].planes), "m": _given(st["opt"].m), "v": _given(st["opt"].v)}
    a, n, k = st["admm"], st["case"]["n"], st["case"]["k"]
    o_t, s_t = P.prox_step(a["o"], a["lam_o"], a["imp"], (3 * n) // 5, a["s"], a["lam_s"], a["amp"], (n * k) // 3)
    P.dual_update_(a["lam_o"], a["o"], o_t)
    P.dual_update_(a["lam_s"], a["s"], s_t)
    P.penalty_grad_(a["g_o"], 5e-4, a["o"], o_t, a["lam_o"])
    P.penalty_grad_(a["g_s"], 5e-4, a["s"], s_t, a["lam_s"])
    ds, kept, lobe_src = P.compact(st["ds"], 0.01, 1.0)
    return {"o_t": o_t, "s_t": s_t, "lam_o": a["lam_o"], "lam_s": a["lam_s"], "g_o": a["g_o"], "g_s": a["g_s"],
            "planes": _given(ds.planes), "lobe_off": ds.lobe_off, "kept": kept, "lobe_src": lobe_src}


# -------------------------------------------------------------------- work ----

def _param_bytes(case):
    eg, ec, ea = (2, 2, 2) if case["half"] else (4, 4, 4)
    k = 0.96 if case["ragged"] else case["k"]
    b = (11 + case["masks"]) * eg
    if case["sh"] >= 0:
        return b + 3 * (case["sh"] + 1) ** 2 * ec
    return b + 3 * ec + k * ((4 + case["masks"]) * ec + 3 * ea) + (4 if case["ragged"] else 0)


def _floats(case):
    k = 0.96 if case["ragged"] else case["k"]
    if case["sh"] >= 0:
        return 11 + case["masks"] + 3 * (case["sh"] + 1) ** 2
    return 14 + case["masks"] + k * (7 + case["masks"])


def _fragments(case):
    """Fragments that pass the alpha test, from the mean footprint: an ellipse of level 2 ln(255 o) around a
    covariance of about (f s / z)^2 + 0.3 px^2, for the share of Gaussians inside the image, and at most 40
    a pixel, after which a pixel of the clustered scenes is opaque on average (counted on the benchmark's batch)."""
    z = 6.0 if case["clustered"] else 4.0
    sizes = [MIXED[i % 4] for i in range(case["views"])] if case["mixed"] else [(case["w"], case["h"])] * case["views"]
    total = 0.0
    for w, h in sizes:
        f = h / 2.0 / math.tan(math.radians(30.0))
        s = f * math.exp(-3.5 + 0.25) / z
        total += min(case["n"] * 0.8 * math.pi * 8.0 * (s * s + 0.3), 40.0 * w * h)
    return total


def work(case):
    kind, n, npix = case["kind"], case["n"], _pixels(case)
    if kind == "loss":  # both images read, the gradient written; two windowed passes of 5 and 3 maps
        return {"bytes": 12.0 * 3 * npix, "flops": 3.0 * npix * (2 * 11 * 2 * 8 + 60)}
    if kind == "adam":  # parameter, both moments read and written, the gradient read
        e = (_param_bytes(case) / _floats(case))
        return {"bytes": n * _floats(case) * (2 * e + 20.0), "flops": 15.0 * n * _floats(case)}
    if kind == "prune":  # scores, values and duals read, selections, duals and gradients written; the scene once
        k = case["k"]
        admm = n * (4 * 3 + 4 * 3 + 8) + n * k * (4 * 5 + 4 * 3 + 8)
        return {"bytes": float(admm + 1.6 * n * _param_bytes(case)), "flops": 40.0 * n * k}
    b = n * _param_bytes(case) + 12.0 * npix
    f = _fragments(case)
    flops = 25.0 * f + 400.0 * n * case["views"]
    if kind == "importance":
        b += 4.0 * n
    if kind in ("grad", "fit") or (kind == "graph" and case["backward"]):
        e = 4.0 * _floats(case) if kind != "grad" or not case["half"] else _param_bytes(case)
        b += n * e + 12.0 * npix
        flops += 45.0 * f + 600.0 * n * case["views"]
    if kind == "fit":
        b += 36.0 * npix
        flops += 3.0 * npix * (2 * 11 * 2 * 8 + 60)
    return {"bytes": float(b), "flops": float(flops)}


# ------------------------------------------------------------------- exact ----

def _ssim_loss(x, y, lam=0.2):
    """(1 - lam) L1 + lam (1 - SSIM), 11-tap Gaussian window of sigma 1.5, zero padding; x, y [3][H][W]."""
    d = torch.arange(11, dtype=torch.float64, device=x.device) - 5.0
    w = torch.exp(-d * d / 4.5)
    w = w / w.sum()

    def win(a):
        a = torch.nn.functional.pad(a, (5, 5, 0, 0))
        a = sum(w[i] * a[:, :, i:i + x.shape[2]] for i in range(11))
        a = torch.nn.functional.pad(a, (0, 0, 5, 5))
        return sum(w[i] * a[:, i:i + x.shape[1], :] for i in range(11))

    mx, my = win(x), win(y)
    sxx, syy, sxy = win(x * x) - mx * mx, win(y * y) - my * my, win(x * y) - mx * my
    s = ((2 * mx * my + 1e-4) * (2 * sxy + 9e-4)) / ((mx * mx + my * my + 1e-4) * (sxx + syy + 9e-4))
    return (1.0 - lam) * (x - y).abs().mean() + lam * (1.0 - s.mean())


def _loss_exact(case, seed, x, y):
    xs = [v.double().requires_grad_(True) for v in R.split_images(x, _cams(case, seed))]
    ys = [v.double() for v in R.split_images(y, _cams(case, seed))]
    loss = sum(_ssim_loss(a, b) for a, b in zip(xs, ys))
    loss.backward()
    return loss.detach(), torch.cat([a.grad.reshape(-1) for a in xs])


def _colour(case, p, off, d):
    """RGB [3][n] of every Gaussian seen along the unit directions d [3][n]."""
    if case["sh"] >= 0:
        x, y, z = d
        Y = [torch.full_like(x, 0.28209479177387814)]
        c1 = 0.48860251190291992
        Y += [-c1 * y, c1 * z, -c1 * x]
        a, b, c = 1.0925484305920792, 0.31539156525252005, 0.54627421529603959
        Y += [a * x * y, -a * y * z, b * (2 * z * z - x * x - y * y), -a * x * z, c * (x * x - y * y)]
        q = 4 * z * z - x * x - y * y
        Y += [-0.59004358992664352 * y * (3 * x * x - y * y), 2.8906114426405538 * x * y * z,
              -0.45704579946446572 * y * q, 0.37317633259011540 * z * (2 * z * z - 3 * x * x - 3 * y * y),
              -0.45704579946446572 * x * q, 1.4453057213202769 * z * (x * x - y * y),
              -0.59004358992664352 * x * (x * x - 3 * y * y)]
        m = p["sh"].shape[0]
        return (torch.stack(Y[:m])[:, None, :] * p["sh"]).sum(0).add(0.5).clamp(min=0.0)
    if case["ragged"]:
        owner = torch.repeat_interleave(torch.arange(case["n"], device=d.device), (off[1:] - off[:-1]).long())
        mu, dd, amp = p["axis"], d[:, owner], p["amp"]
        mu = mu / mu.norm(dim=0)
        e = torch.exp(p["sharp"] * ((mu * dd).sum(0) - 1.0))
        if p["lmask_logit"] is not None:
            e = e * torch.sigmoid(p["lmask_logit"])
        return p["base"].index_add(1, owner, e * amp)
    mu = p["axis"] / p["axis"].norm(dim=1, keepdim=True)
    e = torch.exp(p["sharp"] * ((mu * d).sum(1) - 1.0))
    if p["lmask_logit"] is not None:
        e = e * torch.sigmoid(p["lmask_logit"])
    return p["base"] + (e[:, None, :] * p["amp"]).sum(0)


def _records(case, p, off, cam):
    """(u, v, conic a, b, c, opacity, rgb, depth, kept) of one view in 64 bits."""
    f64 = lambda a: torch.tensor(np.asarray(a, np.float64), device="cuda")
    Rm, t = f64(cam.R), f64(cam.t)
    q = p["quat"] / p["quat"].norm(dim=0)
    w, x, y, z = q
    rot = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                       2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                       2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]).view(3, 3, -1)
    M = rot * torch.exp(p["logscale"])[None]
    c = (Rm[:, :, None] * p["pos"][None]).sum(1) + t[:, None]
    ok = c[2] > cam.znear
    tz = torch.where(ok, c[2], torch.ones_like(c[2]))
    u, v = cam.fx * c[0] / tz + cam.cx, cam.fy * c[1] / tz + cam.cy
    lx, ly = 1.3 * 0.5 * cam.width / cam.fx, 1.3 * 0.5 * cam.height / cam.fy
    xi, eta = (c[0] / tz).clamp(-lx, lx), (c[1] / tz).clamp(-ly, ly)
    T0 = (cam.fx / tz) * Rm[0][:, None] - (cam.fx * xi / tz) * Rm[2][:, None]
    T1 = (cam.fy / tz) * Rm[1][:, None] - (cam.fy * eta / tz) * Rm[2][:, None]
    p0, p1 = (T0[:, None, :] * M).sum(0), (T1[:, None, :] * M).sum(0)
    A, B, C = (p0 * p0).sum(0) + 0.3, (p0 * p1).sum(0), (p1 * p1).sum(0) + 0.3
    det = A * C - B * B
    o = torch.sigmoid(p["op_logit"])
    if p["pmask_logit"] is not None:
        o = o * torch.sigmoid(p["pmask_logit"])
    ok = ok & (o >= 1.0 / 255.0)
    eye = -(Rm.T @ t)
    dv = p["pos"] - eye[:, None]
    rgb = _colour(case, p, off, dv / dv.norm(dim=0))
    return u, v, C / det, -B / det, A / det, o, rgb, c[2].detach().float(), ok


def _composite(case, seed, want_grad, dl_of=None):
    """Images of every view, the importance, and the gradients of the planes for dL/dimage = dl_of(images)."""
    stored, off, _ = _planes(case, seed)
    p = {q: None if t is None else t.double() for q, t in stored.items()}
    leaves = [q for q, t in p.items() if t is not None and t.numel()]
    if want_grad:
        for q in leaves:
            p[q].requires_grad_(True)
    imp = torch.zeros(case["n"], dtype=torch.float64, device="cuda")
    images, recs = [], []
    cams = _cams(case, seed)

    def blend(rec, idx, px, py, flat):
        u, v, a, b, c, o, rgb = rec
        dx, dy = px[:, None] - u[None], py[:, None] - v[None]
        al = (o * torch.exp(-0.5 * (a * dx * dx + 2 * b * dx * dy + c * dy * dy))).clamp(max=0.99)
        al = torch.where(al.detach() >= 1.0 / 255.0, al, torch.zeros_like(al))
        lt = torch.cumsum(torch.log1p(-al), 1)
        live = lt.detach() >= math.log(1e-4)  # the fragment that would take T below 1e-4 is not included
        al = torch.where(live, al, torch.zeros_like(al))
        lt = torch.cumsum(torch.log1p(-al), 1)
        wgt = al * torch.exp(torch.cat([torch.zeros_like(lt[:, :1]), lt[:, :-1]], 1))
        if flat is not None:
            flat.index_add_(0, idx, wgt.detach().sum(0))
        return wgt @ rgb.T

    for cam in cams:
        rec = _records(case, p, off, cam)
        depth, ok = rec[7], rec[8]
        order = torch.argsort(torch.where(ok, depth, torch.full_like(depth, math.inf)), stable=True)[: int(ok.sum())]
        u, v, a, b, c, o, rgb = rec[:7]
        sel = tuple(t[order] for t in (u, v, a, b, c, o)) + (rgb[:, order],)
        recs.append((sel, order))
        grid = torch.arange(cam.width * cam.height, device="cuda")
        step = max(16, int(4.0e7 // max(len(order), 1)))
        out = []
        with torch.no_grad():
            for i in range(0, len(grid), step):
                j = grid[i:i + step]
                out.append(blend([t.detach() for t in sel], order, (j % cam.width) + 0.5, (j // cam.width) + 0.5, imp))
        images.append(torch.cat(out).T.reshape(3, cam.height, cam.width))
    if not want_grad:
        return images, imp, None
    dls = dl_of(images)
    for (sel, order), cam, dl in zip(recs, cams, dls):
        cut = [t.detach().requires_grad_(True) for t in sel]
        grid = torch.arange(cam.width * cam.height, device="cuda")
        step = max(16, int(4.0e7 // max(len(order), 1)))
        d = dl.reshape(3, -1).T
        for i in range(0, len(grid), step):
            j = grid[i:i + step]
            blend(cut, order, (j % cam.width) + 0.5, (j // cam.width) + 0.5, None).backward(d[i:i + step])
        torch.autograd.backward(sel, [t.grad for t in cut], retain_graph=True)
    grads = {q: p[q].grad if p[q].grad is not None else torch.zeros_like(p[q]) for q in leaves}
    return images, imp, grads


def _compact_exact(case, seed, p):
    """The post-processing by its definition: what is kept, folded masks, compensated base colours."""
    n, k = case["n"], case["k"]
    d = {q: None if t is None else t.double() for q, t in p.items()}
    pm = d["pmask_logit"]
    o = torch.sigmoid(d["op_logit"])
    keep = (o if pm is None else o * torch.sigmoid(pm)) >= 0.01
    idx = torch.nonzero(keep)[:, 0]
    lk = (d["sharp"] >= 1.0) & keep[None]
    m = torch.ones_like(d["sharp"]) if d["lmask_logit"] is None else torch.sigmoid(d["lmask_logit"])
    s = d["sharp"]
    mean = torch.where(s == 0, torch.ones_like(s), -torch.expm1(-2 * s) / (2 * s))
    base = d["base"] + ((m * mean * (d["sharp"] < 1.0))[:, None] * d["amp"]).sum(0)
    op = d["op_logit"] if pm is None else -torch.logsumexp(torch.stack([-d["op_logit"], -pm, -d["op_logit"] - pm]), 0)
    g, l = torch.nonzero(lk.T, as_tuple=True)  # Gaussian-major
    amp = m[:, None] * d["amp"]
    return {"pos": d["pos"][:, idx], "logscale": d["logscale"][:, idx], "quat": d["quat"][:, idx], "op_logit": op[idx],
            "base": base[:, idx], "axis": d["axis"][l, :, g].T, "sharp": s[l, g], "amp": amp[l, :, g].T}


def exact(case, seed):
    kind = case["kind"]
    if kind == "loss":
        loss, g = _loss_exact(case, seed, *_image_pair(case, seed))
        return {"loss": loss, "grad": g}
    if kind == "adam":
        p, gmv = _adam_inputs(case, seed)
        out = {"planes": {}, "m": {}, "v": {}}
        f = lambda v: float(np.float32(v))  # the settings as the optimiser receives them
        b1, b2, eps, t = f(0.9), f(0.999), f(1e-15), 1000
        for q, (g, m, v) in gmv.items():
            g = g.double()
            m1 = b1 * m.double() + (1 - b1) * g
            v1 = b2 * v.double() + (1 - b2) * g * g
            out["m"][q], out["v"][q] = m1, v1
            out["planes"][q] = p[q].double() - f(T.DEFAULT_LR[q]) * (m1 / (1 - b1 ** t)) / ((v1 / (1 - b2 ** t)).sqrt() + eps)
        return {a: _given(b) for a, b in out.items()}
    if kind == "prune":
        p, _, _ = _planes(case, seed)
        a = {q: t.double() for q, t in _admm_inputs(case, p, seed).items()}
        keep = torch.zeros(case["n"], dtype=torch.bool, device="cuda")
        keep[torch.sort(a["imp"], descending=True, stable=True).indices[: (3 * case["n"]) // 5]] = True
        o_t = torch.where(keep, a["o"] + a["lam_o"], torch.zeros_like(a["o"]))
        lam_o = a["lam_o"] + (a["o"] - o_t)
        # the lobe selection ranks 32-bit scores: what follows from it has no 64-bit value here
        return {"o_t": o_t, "s_t": None, "lam_o": lam_o, "lam_s": None,
                "g_o": a["g_o"] + float(np.float32(5e-4)) * ((a["o"] - o_t) + lam_o), "g_s": None,
                "planes": _compact_exact(case, seed, p), "lobe_off": None, "kept": None, "lobe_src": None}
    if case["n"] * float(_pixels(case)) > EXACT_PRODUCTS:
        return None
    cams = _cams(case, seed)
    if kind == "view":
        return {"images": _composite(case, seed, False)[0]}
    if kind == "importance":
        images, imp, _ = _composite(case, seed, False)
        return {"images": images, "importance": imp}
    if kind == "graph" and not case["backward"]:
        return {"images": _composite(case, seed, False)[0]}
    if kind == "fit":
        y = _image_pair(case, seed)[1]
        kept = {}

        def dl_of(images):
            kept["loss"], dl = _loss_exact(case, seed, torch.cat([x.reshape(-1) for x in images]), y)
            return R.split_images(dl, cams)

        images, _, grads = _composite(case, seed, True, dl_of)
        return {"images": images, "loss": kept["loss"], "grads": grads}
    w = R.split_images(_weights(case, seed, _pixels(case)).double(), cams)
    images, _, grads = _composite(case, seed, True, lambda _: w)
    return {"images": images, "grads": grads}
