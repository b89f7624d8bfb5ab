"""Performance cases of the library: what its users have it do, through the
public Python entry points, over the range of sizes, types and options.

A case is a dict of plain values; `kind` names the path:
  filter        Filter.run on one resident cube (noise level estimated on the
                GPU unless `rms` is given)
  batch         batch() on a prepared list of uneven cubes
  quality       quality() of an original and a filtered cube with a model
  smooth        smooth(), box or Gaussian, axis-aligned or rotated
  wavelet       wavelet_denoise / wavelet_forward / wavelet_inverse
  infer, train  the learned surrogate: one prediction, one training step

Inputs are synthetic H I cubes: noise of rms 1 plus exponential disks (peak
S/N 10) on rotation curves and faint one-pixel tails, drawn on the GPU from
the seed alone.  `exact` computes each result in 64 bits with plain torch.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_1609_03782_amd as ig
from paper_1609_03782_amd import surrogate

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
MAX_VOXELS = 512 ** 3
MAX_VOXEL_STEPS = 50 * MAX_VOXELS
DEPTH = 8          # layers of the reference surrogate
WIDTH = 32         # its hidden channels


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # one small cube (a cut-out around one galaxy): launches and latency count
        {"name": "filter_small", "kind": "filter", "nx": 64, "ny": 64, "nz": 32, "cond": "pm_exp", "dtype": "f32",
         "K": 2.0, "tau": 0.0625, "C": 1.0, "n_iter": 10, "rms": 0.0},
        # interactive use: about 5e6 voxels of no particular size, the paper's
        # default parameters (intensity conductance, 20 steps)
        {"name": "filter_interactive", "kind": "filter", "nx": 187, "ny": 181, "nz": 149, "cond": "intensity",
         "dtype": "f32", "K": 1.5, "tau": 0.0325, "C": 5.0, "n_iter": 20, "rms": 0.0},
        # a whole survey cube, the headline workload of the benchmark
        {"name": "filter_survey", "kind": "filter", "nx": 512, "ny": 512, "nz": 512, "cond": "pm_exp", "dtype": "f32",
         "K": 2.0, "tau": 0.0625, "C": 1.0, "n_iter": 50, "rms": 0.0},
        # a ragged cube kept in 16 bits to halve its memory
        {"name": "filter_half", "kind": "filter", "nx": 300, "ny": 400, "nz": 490, "cond": "pm_exp", "dtype": "bf16",
         "K": 2.0, "tau": 0.0625, "C": 1.0, "n_iter": 50, "rms": 0.0},
        # a wide mosaic of few channels, more than one tile in x, rational weights
        {"name": "filter_wide", "kind": "filter", "nx": 1000, "ny": 700, "nz": 61, "cond": "pm_rational",
         "dtype": "f32", "K": 2.0, "tau": 0.0625, "C": 1.0, "n_iter": 20, "rms": 1.0},
        # a catalogue of cut-outs, each with its own size, K and step count, in one call
        {"name": "batch_catalogue", "kind": "batch", "count": 96, "lo": 32, "hi": 256, "hi_z": 160, "plan": 4},
        # the quality curve of a filtered survey cube: 46 mask thresholds, 0 to 4.5 rms
        {"name": "quality_curve", "kind": "quality", "nx": 512, "ny": 512, "nz": 512, "thresholds": 46, "model": True,
         "roi": False},
        # pre-smoothing before the wavelet denoiser (FWHM 5)
        {"name": "smooth_gauss", "kind": "smooth", "nx": 512, "ny": 512, "nz": 512, "shape": "gauss", "sx": 5.0,
         "sy": 5.0, "sz": 5.0, "ax": 0.0, "ay": 0.0, "az": 0.0},
        # an elongated beam at an angle: the rotated kernel has no separable form
        {"name": "smooth_rotated", "kind": "smooth", "nx": 360, "ny": 350, "nz": 290, "shape": "gauss", "sx": 2.0,
         "sy": 3.0, "sz": 3.0, "ax": 10.0, "ay": 20.0, "az": 30.0},
        # the paper's wavelet denoiser: Haar, three levels, noise level estimated
        {"name": "wavelet_haar", "kind": "wavelet", "nx": 512, "ny": 512, "nz": 512, "wavelet": "haar", "levels": 3,
         "op": "denoise", "rms": 0.0},
        # a whole prediction of the learned surrogate on a ragged cube
        {"name": "surrogate_infer", "kind": "infer", "nx": 360, "ny": 360, "nz": 150},
        # one training step as the surrogate is trained: four 96^3 cubes
        {"name": "surrogate_train", "kind": "train", "n": 96, "batch": 4},
    ]


def _logint(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_shape(rng, lo, hi, limit):
    nx, ny, nz = _logint(rng, lo, hi), _logint(rng, lo, hi), _logint(rng, lo, min(hi, 512))
    while nx * ny * nz > limit:
        nx, ny, nz = max(lo, nx * 4 // 5), max(lo, ny * 4 // 5), max(lo, nz * 4 // 5)
    if rng.random() < 0.4:   # round sizes are as common as odd ones
        nx = max(8, nx - nx % 8)
    return {"nx": nx, "ny": ny, "nz": nz}


def draw(rng):
    kind = rng.choice(["filter", "filter", "filter", "batch", "quality", "smooth", "smooth", "wavelet", "wavelet",
                       "infer", "train"])
    if kind == "filter":
        c = {"kind": kind, **_draw_shape(rng, 24, 1024, MAX_VOXELS)}
        c["cond"] = rng.choice(["pm_exp", "pm_exp", "intensity", "pm_rational"])
        c["dtype"] = rng.choice(["f32", "f32", "bf16", "f16"])
        c["K"] = round(rng.uniform(1.0, 3.0), 2)
        c["tau"], c["C"] = (0.0325, 5.0) if c["cond"] == "intensity" else (0.0625, 1.0)
        c["n_iter"] = min(rng.randint(5, 60), max(1, MAX_VOXEL_STEPS // (c["nx"] * c["ny"] * c["nz"])))
        c["rms"] = rng.choice([0.0, 1.0])
        return c
    if kind == "batch":
        hi = rng.randint(64, 256)
        return {"kind": kind, "count": rng.randint(8, 96), "lo": rng.randint(16, 48), "hi": hi,
                "hi_z": min(hi, 160), "plan": rng.randint(1, 1000)}
    if kind == "quality":
        return {"kind": kind, **_draw_shape(rng, 48, 1024, MAX_VOXELS), "thresholds": rng.choice([1, 3, 8, 19, 46]),
                "model": rng.random() < 0.7, "roi": rng.random() < 0.4}
    if kind == "smooth":
        rot = rng.random() < 0.5
        c = {"kind": kind, **_draw_shape(rng, 32, 1024, 360 * 350 * 290 if rot else MAX_VOXELS)}
        box = not rot and rng.random() < 0.4
        c["shape"] = "box" if box else "gauss"
        for a in "xyz":
            c["s" + a] = float(rng.choice([3, 5, 7])) if box else round(rng.uniform(1.5, 3.0 if rot else 5.0), 1)
            c["a" + a] = round(rng.uniform(5.0, 60.0), 1) if rot else 0.0
        return c
    if kind == "wavelet":
        return {"kind": kind, **_draw_shape(rng, 32, 1024, MAX_VOXELS), "wavelet": rng.choice(["haar", "legall53"]),
                "levels": rng.randint(1, 4), "op": rng.choice(["denoise", "denoise", "forward", "inverse"]),
                "rms": rng.choice([0.0, 1.0])}
    if kind == "infer":
        return {"kind": kind, **_draw_shape(rng, 24, 512, 360 * 360 * 150)}
    return {"kind": "train", "n": rng.randint(24, 96), "batch": rng.randint(1, 4)}


# ------------------------------------------------------------------ inputs
def _paint(em, rnd, galaxies, tails):
    """Adds exponential disks and quadratic tails to the emission cube em."""
    nz, ny, nx = em.shape
    for _ in range(galaxies):
        h = rnd.uniform(3.0, max(4.0, min(nx, ny) / 13.0))
        xc, yc, v0 = rnd.uniform(0.1, 0.9) * nx, rnd.uniform(0.1, 0.9) * ny, rnd.uniform(0.3, 0.7) * nz
        inc, pa = math.radians(rnd.uniform(30.0, 75.0)), math.radians(rnd.uniform(0.0, 360.0))
        xa, xb = max(0, int(xc - 7 * h)), min(nx, int(xc + 7 * h) + 2)
        ya, yb = max(0, int(yc - 7 * h)), min(ny, int(yc + 7 * h) + 2)
        x = torch.arange(xa, xb, device=DEV, dtype=torch.float32)[None, :] - xc
        y = torch.arange(ya, yb, device=DEV, dtype=torch.float32)[:, None] - yc
        xd = x * math.cos(pa) + y * math.sin(pa)
        yd = (y * math.cos(pa) - x * math.sin(pa)) / math.cos(inc)
        R = torch.sqrt(xd * xd + yd * yd)
        v = v0 + 0.25 * nz * torch.sin(0.5 * math.pi * torch.clamp(R / (2 * h), max=1.0)) * xd / torch.clamp(R, min=1e-6)
        za, zb = max(0, int(v0 - 0.25 * nz - 6)), min(nz, int(v0 + 0.25 * nz + 8))
        z = torch.arange(za, zb, device=DEV, dtype=torch.float32)[:, None, None]
        em[za:zb, ya:yb, xa:xb] += 10.0 * torch.exp(-R / h) * torch.exp(-0.5 * (z - v) ** 2)
    for _ in range(tails):
        p = [[rnd.uniform(0.1, 0.9) * s for s in (nx, ny, nz)] for _ in range(3)]
        u = torch.linspace(0.0, 1.0, 4 * max(nx, ny, nz), device=DEV, dtype=torch.float64)[:, None]
        q = torch.tensor(p, device=DEV, dtype=torch.float64)
        at = torch.round((1 - u) ** 2 * q[0] + 2 * (1 - u) * u * q[1] + u ** 2 * q[2]).long()
        em.view(-1)[torch.unique((at[:, 2] * ny + at[:, 1]) * nx + at[:, 0])] += rnd.uniform(0.5, 1.5)


def _cube(shape, seed, galaxies=None, tails=None):
    """(noisy cube, emission), FP32, both from the seed alone."""
    rnd = random.Random(seed)
    if galaxies is None:
        galaxies = max(1, min(8, shape[0] * shape[1] * shape[2] // 2 ** 22))
    em = torch.zeros(shape, device=DEV, dtype=torch.float32)
    _paint(em, rnd, galaxies, 1 if tails is None else tails)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    x = torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)
    return x.add_(em), em


def _neighbour_mean(x, steps=1):
    """Explicit linear diffusion steps in plain torch (a smoothed cube)."""
    for _ in range(steps):
        acc = torch.zeros_like(x)
        for a in range(3):
            d = (x.narrow(a, 1, x.shape[a] - 1) - x.narrow(a, 0, x.shape[a] - 1)) * 0.12
            acc.narrow(a, 0, x.shape[a] - 1).add_(d)
            acc.narrow(a, 1, x.shape[a] - 1).sub_(d)
        x = x + acc
    return x


def _shape(case):
    return (case["nz"], case["ny"], case["nx"])


def _batch_items(case):
    rnd = random.Random(case["plan"])
    items = []
    for k in range(case["count"]):
        nx, ny = _logint(rnd, case["lo"], case["hi"]), _logint(rnd, case["lo"], case["hi"])
        nz = _logint(rnd, case["lo"], max(case["lo"], case["hi_z"]))
        items.append(((nz, ny, nx), round(rnd.uniform(1.5, 3.0), 3), rnd.randint(20, 80)))
    return items


def _batch_inputs(case, seed):
    """One allocation for all cubes (each starting at a multiple of 64 voxels)
    and the cubes' views in it."""
    items = _batch_items(case)
    starts, total = [], 0
    for shape, _, _ in items:
        starts.append(total)
        total += -(-shape[0] * shape[1] * shape[2] // 64) * 64
    flat = torch.zeros(total, device=DEV, dtype=torch.float32)
    views = []
    for k, ((shape, _, _), at) in enumerate(zip(items, starts)):
        v = flat[at:at + shape[0] * shape[1] * shape[2]].view(shape)
        v.copy_(_cube(shape, seed * 1009 + k, galaxies=1, tails=k % 2)[0])
        views.append(v)
    return items, flat, views, starts


def _weights(seed):
    """Weights of a network as training leaves it: hidden layers at the He
    scale, a small last layer; per layer W [27][c_in][c_out] then b."""
    g = torch.Generator()
    g.manual_seed(seed)
    Ws, bs = [], []
    for l in range(DEPTH):
        cin, cout = (1 if l == 0 else WIDTH), (1 if l == DEPTH - 1 else WIDTH)
        sd = 0.02 if l == DEPTH - 1 else math.sqrt(2.0 / (27.0 * cin))
        Ws.append(torch.randn((27, cin, cout), generator=g) * sd)
        bs.append(torch.randn((cout,), generator=g) * 0.05)
    return Ws, bs


def _flat_weights(Ws, bs):
    return torch.cat([torch.cat([W.reshape(-1), b]) for W, b in zip(Ws, bs)]).numpy()


def _train_pairs(case, seed):
    n = case["n"]
    xs = [_cube((n, n, n), seed * 1009 + k, galaxies=1, tails=k % 2)[0] for k in range(case["batch"])]
    return xs, [_neighbour_mean(x, 10) for x in xs]


def _thresholds(case):
    k = case["thresholds"]
    return [3.0] if k == 1 else [4.5 * j / (k - 1) for j in range(k)]


def _roi(case):
    if not case["roi"]:
        return None
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    return (nx // 7, nx - nx // 9, ny // 8, ny - ny // 6, nz // 10, nz - nz // 12)


def _wavelet_t(case):
    t = (0.5, 0.8, 1.1, 1.3) if case["wavelet"] == "haar" else (1.0, 1.4, 1.7, 1.9)
    return t[:case["levels"]]


# ------------------------------------------------------------------ one case
def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "filter":
        s["x"] = _cube(_shape(case), seed)[0].to(DTYPES[case["dtype"]])
        s["out"] = torch.empty_like(s["x"])
        s["f"] = ig.Filter(_shape(case), K=case["K"], tau=case["tau"], n_iter=case["n_iter"], C=(case["C"],) * 3,
                           rms=case["rms"] or None, cond=case["cond"], dtype=case["dtype"])
    elif kind == "batch":
        items, s["flat"], views, starts = _batch_inputs(case, seed)
        s["out"] = torch.zeros_like(s["flat"])
        outs = [s["out"][a:a + v.numel()].view(v.shape) for a, v in zip(starts, views)]
        s["batch"] = ig.batch_prepare([(v, o, {"K": K, "tau": 0.0625, "n_iter": n, "cond": "pm_exp"})
                                       for v, o, (_, K, n) in zip(views, outs, items)])
    elif kind == "quality":
        s["x"], s["model"] = _cube(_shape(case), seed)
        s["y"] = _neighbour_mean(s["x"])
    elif kind == "smooth":
        s["x"] = _cube(_shape(case), seed)[0]
        s["out"], s["work"] = torch.empty_like(s["x"]), torch.empty_like(s["x"])
    elif kind == "wavelet":
        s["x"] = _neighbour_mean(_cube(_shape(case), seed)[0])
        s["out"] = torch.empty_like(s["x"])
    else:
        Ws, bs = _weights(seed)
        s["net"] = surrogate.Surrogate(depth=DEPTH, width=WIDTH, lr=3e-4, seed=1)
        s["net"].set_weights(_flat_weights(Ws, bs))
        if kind == "infer":
            s["x"] = _cube(_shape(case), seed)[0]
            s["out"] = torch.empty_like(s["x"])
        else:
            s["xs"], s["ts"] = _train_pairs(case, seed)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "filter":
        return s["f"].run(s["x"], s["out"])
    if kind == "batch":
        ig.batch(s["batch"])
        return s["out"]
    if kind == "quality":
        r = ig.quality(s["x"], s["y"], s["model"] if case["model"] else None, roi=_roi(case), thr_f=_thresholds(case))
        return {k: np.asarray(v) for k, v in r.items() if v is not None and v != []}
    if kind == "smooth":
        return ig.smooth(s["x"], case["shape"], (case["sx"], case["sy"], case["sz"]),
                         (case["ax"], case["ay"], case["az"]), out=s["out"], work=s["work"])
    if kind == "wavelet":
        if case["op"] == "denoise":
            return ig.wavelet_denoise(s["x"], case["wavelet"], case["levels"], _wavelet_t(case), rms=case["rms"],
                                      out=s["out"])
        fn = ig.wavelet_forward if case["op"] == "forward" else ig.wavelet_inverse
        return fn(s["x"], case["wavelet"], case["levels"], out=s["out"])
    if kind == "infer":
        return s["net"].infer(s["x"], out=s["out"])
    loss = s["net"].train_step(s["xs"], s["ts"])
    return loss, s["net"].get_grads()


# ------------------------------------------------------------------ work
def _half_widths(case):
    if case["shape"] == "box":
        return [int(case["s" + a]) // 2 for a in "xyz"]
    sig = [case["s" + a] * 0.42466090014400953 for a in "xyz"]
    if not (case["ax"] or case["ay"] or case["az"]):
        return [int(math.floor(3 * v + 0.5)) for v in sig]
    R = _rotation(case)
    return [int(math.floor(3 * math.sqrt(sum((R[i][j] * sig[j]) ** 2 for j in range(3))) + 0.5)) for i in range(3)]


def _rotation(case):
    cx, cy, cz = (math.cos(math.radians(case["a" + a])) for a in "xyz")
    sx, sy, sz = (math.sin(math.radians(case["a" + a])) for a in "xyz")
    return [[cz * cy, cz * sy * sx - sz * cx, cz * sy * cx + sz * sx],
            [sz * cy, sz * sy * sx + cz * cx, sz * sy * cx - cz * sx],
            [-sy, cy * sx, cy * cx]]


# operations of one voxel and step: three edge terms and the update
STEP_OPS = {"pm_exp": 3 * 6 + 6, "pm_rational": 3 * 6 + 6, "intensity": 3 * 2 + 11}
NET_FLOPS = 2 * 27 * (WIDTH + (DEPTH - 2) * WIDTH * WIDTH + WIDTH)   # one prediction, per voxel


def work(case):
    kind = case["kind"]
    if kind == "batch":
        vox = vi = 0
        for shape, _, n in _batch_items(case):
            v = shape[0] * shape[1] * shape[2]
            vox, vi = vox + v, vi + v * n
        return {"bytes": 8.0 * vox, "flops": float(STEP_OPS["pm_exp"] * vi)}
    if kind == "train":
        v = case["batch"] * case["n"] ** 3
        return {"bytes": 8.0 * v, "flops": float(v * (3 * NET_FLOPS - 2 * 27 * WIDTH))}
    v = case["nx"] * case["ny"] * case["nz"]
    if kind == "filter":
        size = 4 if case["dtype"] == "f32" else 2
        return {"bytes": 2.0 * size * v, "flops": float(v * case["n_iter"] * STEP_OPS[case["cond"]])}
    if kind == "quality":
        return {"bytes": (12.0 if case["model"] else 8.0) * v, "flops": 6.0 * v}
    if kind == "smooth":
        r = _half_widths(case)
        if case["ax"] or case["ay"] or case["az"]:
            taps = (2 * r[0] + 1) * (2 * r[1] + 1) * (2 * r[2] + 1)
        else:
            taps = sum(2 * k + 1 for k in r)
        return {"bytes": 8.0 * v, "flops": 2.0 * taps * v}
    if kind == "wavelet":
        per = 3 * (1.5 if case["wavelet"] == "haar" else 3.0)
        return {"bytes": 8.0 * v, "flops": per * v * (2 if case["op"] == "denoise" else 1)}
    return {"bytes": 8.0 * v, "flops": float(NET_FLOPS) * v}


# ------------------------------------------------------------------ 64 bits
def _filter64(x, cond, K, tau, C, n_iter, rms):
    store = x.dtype   # 16-bit storage rounds after every step
    x = x.double()
    rho = rms if rms > 0 else float(torch.sqrt((x * x).mean()))
    f32 = lambda v: float(torch.tensor(v, dtype=torch.float32))   # noqa: E731  the entry points take these as FP32
    kr, tc = f32(K) * rho, f32(tau) * f32(C)
    for _ in range(n_iter):
        acc = torch.zeros_like(x)
        for a in range(3):
            m = x.shape[a] - 1
            if m < 1:
                continue
            d = x.narrow(a, 1, m) - x.narrow(a, 0, m)
            if cond == "pm_exp":
                e = d * torch.exp(-(d / kr) ** 2).mul_(tc)
            elif cond == "pm_rational":
                e = d * tc / (1.0 + (d / kr) ** 2)
            else:
                e = d * f32(C)
            acc.narrow(a, 0, m).add_(e)
            acc.narrow(a, 1, m).sub_(e)
        x = x + (acc * f32(tau) / (1.0 + (x / kr) ** 2) if cond == "intensity" else acc)
        if store != torch.float32:
            x = x.to(store).double()
    return x


def _quality64(case, seed):
    x, model = _cube(_shape(case), seed)
    y = _neighbour_mean(x).double()
    x, model = x.double(), model.double()
    rms_o, rms_f = float(torch.sqrt((x * x).mean())), float(torch.sqrt((y * y).mean()))
    r = _roi(case)
    if r is not None:
        x, y, model = (t[r[4]:r[5], r[2]:r[3], r[0]:r[1]] for t in (x, y, model))
    mo = x >= 3.0 * rms_o
    S_oo, N_o, S_m = float(x[mo].sum()), int(mo.sum()), float(model.sum())
    S_of, N_f, S_mf, F, sF, FM, sFM = [], [], [], [], [], [], []
    s_oo = math.sqrt(N_o) * rms_o
    for t in _thresholds(case):
        m = y >= t * rms_f
        S, N = float(torch.where(m, x, 0.0).sum()), int(m.sum())
        s_of = math.sqrt(N) * rms_f
        S_of.append(S)
        N_f.append(N)
        F.append(abs(S) / abs(S_oo))
        sF.append(math.sqrt(s_of ** 2 / S_oo ** 2 + S ** 2 * s_oo ** 2 / S_oo ** 4))
        if case["model"]:
            S_mf.append(float(torch.where(m, model, 0.0).sum()))
            FM.append(abs(S_mf[-1]) / abs(S_m))
            sFM.append(s_of / abs(S_m))
    out = {"rms_o": rms_o, "rms_f": rms_f, "S_oo": S_oo, "N_o": N_o, "n_roi": x.numel(), "S_of": S_of, "N_f": N_f,
           "F": F, "sigma_F": sF}
    if case["model"]:
        out.update({"S_m": S_m, "S_mf": S_mf, "F_M": FM, "sigma_FM": sFM})
    return {k: np.asarray(v) for k, v in out.items()}


def _smooth64(case, x):
    x = x.double()
    r = _half_widths(case)
    one = torch.ones_like(x)
    if not (case["ax"] or case["ay"] or case["az"]):
        num = x
        for a, (k, ax) in enumerate(zip(r[::-1], "zyx")):
            sig = case["s" + ax] * 0.42466090014400953
            n = x.shape[a]
            line = torch.zeros(n, device=DEV, dtype=torch.float64)
            acc = torch.zeros_like(x)
            for d in range(-k, k + 1):
                if abs(d) >= n:
                    continue
                w = 1.0 if case["shape"] == "box" else math.exp(-d * d / (2 * sig * sig))
                to, m = max(0, -d), n - abs(d)
                acc.narrow(a, to, m).add_(num.narrow(a, max(0, d), m), alpha=w)
                line[to:to + m] += w
            num = acc / line.view([n if b == a else 1 for b in range(3)])
        return num
    R, sig = _rotation(case), [case["s" + a] * 0.42466090014400953 for a in "xyz"]
    num, den = torch.zeros_like(x), torch.zeros_like(x)
    nz, ny, nx = x.shape
    for dz in range(-r[2], r[2] + 1):
        for dy in range(-r[1], r[1] + 1):
            for dx in range(-r[0], r[0] + 1):
                if abs(dz) >= nz or abs(dy) >= ny or abs(dx) >= nx:
                    continue
                d = (dx, dy, dz)
                u = [sum(R[i][j] * d[i] for i in range(3)) for j in range(3)]
                w = math.exp(-sum(u[j] ** 2 / (2 * sig[j] ** 2) for j in range(3)))
                to = tuple(slice(max(0, -o), n - max(0, o)) for o, n in ((dz, nz), (dy, ny), (dx, nx)))
                at = tuple(slice(max(0, o), n + min(0, o)) for o, n in ((dz, nz), (dy, ny), (dx, nx)))
                num[to].add_(x[at], alpha=w)
                den[to].add_(one[at], alpha=w)
    return num / den


def _lift64(x, axis, kind, inverse):
    n = x.shape[axis]
    if n < 2:
        return x
    ne, no = (n + 1) // 2, n // 2
    cut = lambda t, a, m: t.narrow(axis, a, m)   # noqa: E731
    if inverse:
        ev, od = cut(x, 0, ne).clone(), cut(x, ne, no).clone()
    else:
        at = torch.arange(n, device=x.device)
        ev, od = x.index_select(axis, at[0::2]), x.index_select(axis, at[1::2])

    def predict(e):
        if kind == "haar":
            return cut(e, 0, no)
        right = torch.cat([cut(e, 1, ne - 1), cut(e, ne - 1, 1)], axis)
        return (cut(e, 0, no) + cut(right, 0, no)) * 0.5

    def update(d):
        if kind == "haar":
            u = d * 0.5
            return u if ne == no else torch.cat([u, torch.zeros_like(cut(u, 0, 1))], axis)
        left = torch.cat([cut(d, 0, 1), d], axis)
        right = d if ne == no else torch.cat([d, cut(d, no - 1, 1)], axis)
        return (cut(left, 0, ne) + right) * 0.25

    if not inverse:
        od = od - predict(ev)
        return torch.cat([ev + update(od), od], axis)
    ev = ev - update(od)
    od = od + predict(ev)
    out = torch.empty_like(x)
    at = torch.arange(n, device=x.device)
    out.index_copy_(axis, at[0::2], ev)
    out.index_copy_(axis, at[1::2], od)
    return out


def _wavelet64(case, x):
    x = x.double()
    rms = case["rms"] if case["rms"] > 0 else float(torch.sqrt((x * x).mean()))
    kind, L, t = case["wavelet"], case["levels"], _wavelet_t(case)
    boxes = [tuple(x.shape)]
    for _ in range(L):
        boxes.append(tuple((n + 1) // 2 for n in boxes[-1]))
    c = x.clone()
    if case["op"] != "inverse":
        for l in range(L):
            b = tuple(slice(0, n) for n in boxes[l])
            for a in (2, 1, 0):
                c[b] = _lift64(c[b].clone(), a, kind, False)
    if case["op"] == "denoise":
        level = torch.full(x.shape, L, dtype=torch.uint8, device=DEV)   # the last box shares the last threshold
        for l in range(L - 1, -1, -1):
            keep = level[tuple(slice(0, n) for n in boxes[l + 1])].clone()
            level[tuple(slice(0, n) for n in boxes[l])] = l + 1
            level[tuple(slice(0, n) for n in boxes[l + 1])] = keep
        for l in range(L):
            c[(level == l + 1) & (c.abs() < t[l] * rms)] = 0.0
    if case["op"] != "forward":
        for l in range(L - 1, -1, -1):
            b = tuple(slice(0, n) for n in boxes[l])
            for a in (0, 1, 2):
                c[b] = _lift64(c[b].clone(), a, kind, True)
    return (c, rms) if case["op"] == "denoise" else c


def _conv64(a, W, b):
    """3x3x3 convolution of a (nz, ny, nx, c_in), zero padding, as 27 products."""
    nz, ny, nx, cin = a.shape
    p = torch.nn.functional.pad(a, (0, 0, 1, 1, 1, 1, 1, 1))
    out = b.expand(nz * ny * nx, -1)
    for t in range(27):
        dz, dy, dx = t // 9, (t // 3) % 3, t % 3
        out = out + p[dz:dz + nz, dy:dy + ny, dx:dx + nx].reshape(-1, cin) @ W[t]
    return out.view(nz, ny, nx, -1)


def _net64(x, Ws, bs):
    a = x[..., None]
    for l, (W, b) in enumerate(zip(Ws, bs)):
        a = _conv64(a, W, b)
        if l < len(Ws) - 1:
            a = torch.nn.functional.gelu(a)
    return x + a[..., 0]


def exact(case, seed):
    kind = case["kind"]
    if kind == "filter":
        x = _cube(_shape(case), seed)[0].to(DTYPES[case["dtype"]])
        return _filter64(x, case["cond"], case["K"], case["tau"], case["C"], case["n_iter"], case["rms"])
    if kind == "batch":
        items, flat, views, starts = _batch_inputs(case, seed)
        out = torch.zeros_like(flat, dtype=torch.float64)
        for v, at, (_, K, n) in zip(views, starts, items):
            out[at:at + v.numel()] = _filter64(v, "pm_exp", K, 0.0625, 1.0, n, 0.0).view(-1)
        return out
    if kind == "quality":
        return _quality64(case, seed)
    if kind == "smooth":
        return _smooth64(case, _cube(_shape(case), seed)[0])
    if kind == "wavelet":
        return _wavelet64(case, _neighbour_mean(_cube(_shape(case), seed)[0]))
    Ws, bs = _weights(seed)
    Ws, bs = [W.to(DEV).double() for W in Ws], [b.to(DEV).double() for b in bs]
    if kind == "infer":
        x = _cube(_shape(case), seed)[0].double()
        out = torch.empty_like(x)
        with torch.no_grad():   # in runs of planes, each with the planes its outputs depend on
            for z in range(0, x.shape[0], 48):
                a, b = max(0, z - DEPTH), min(x.shape[0], z + 48 + DEPTH)
                e = min(x.shape[0], z + 48)
                out[z:e] = _net64(x[a:b], Ws, bs)[z - a:e - a]
        return out
    xs, ts = _train_pairs(case, seed)
    for p in Ws + bs:
        p.requires_grad_(True)
    total = sum(x.numel() for x in xs)
    loss = 0.0
    for x, t in zip(xs, ts):
        part = ((_net64(x.double(), Ws, bs) - t.double()) ** 2).sum() / total
        part.backward()
        loss += float(part)
    return loss, torch.cat([torch.cat([W.grad.reshape(-1), b.grad]) for W, b in zip(Ws, bs)]).cpu().numpy()
