"""Performance cases of the cavity library: the calls a user's program makes,
over the sizes it makes them at.

Every case goes through the package's Python binding with the library's
default execution options, the way README.md and the workflow modules
(configs, flowmap, warmstart) use it: a handle is created and its start state
loaded in `prepare`; `run` advances it and fetches what the program wants to
see.  A lattice handle keeps its state from pass to pass, as a running
simulation does.

`exact` states the same quantities in 64-bit torch and NumPy.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2211_05009_amd import lbm

U_LID = 0.1
DEV = "cuda"

# ------------------------------------------------------------------ the cases


def _cavity(name, nx, ny, re, dtype, wall, steps):
    return {"name": name, "kind": "cavity", "nx": nx, "ny": ny, "re": re, "dtype": dtype,
            "wall": wall, "steps": steps}


def listed():
    return [
        # the 64 x 64, Re 100 validation cavity between two monitor points
        _cavity("cavity-64-f64", 64, 64, 100.0, "f64", "bounce-back", 100),
        # a short call on the production lattice: 20 steps, then the fields
        # (an animation, a coupling step)
        _cavity("call-500-f32", 500, 500, 8000.0, "f32s", "bounce-back", 20),
        # the production lattice, a stretch of a long run
        _cavity("cavity-500-f32", 500, 500, 8000.0, "f32s", "bounce-back", 1000),
        # the tall production lattice in FP64 (the study to tight thresholds)
        _cavity("cavity-500x1000-f64", 500, 1000, 4000.0, "f64", "bounce-back", 500),
        # the large lattice, beyond the caches
        _cavity("cavity-4096-f32", 4096, 4096, 1e4, "f32s", "bounce-back", 100),
        # the paper's own walls on the Table 1 lattice
        _cavity("nee-257-f64", 257, 257, 1000.0, "f64", "nee", 500),
        # the 25-cavity Re x Ar sweep as one batch, then each cavity's canvas
        {"name": "sweep-25-f32", "kind": "batch", "nx": 500, "cavities": 25, "re_lo": 4000.0,
         "re_hi": 8000.0, "dtype": "f32s", "steps": 1000},
        # the lid-driven box, then its fields on the host
        {"name": "box-192-f64", "kind": "box", "nx": 192, "ny": 192, "nz": 192, "re": 1000.0,
         "dtype": "f64", "steps": 300},
        # the warm-start network on the steady sweep's batch
        {"name": "predict-8", "kind": "predict", "n": 8},
        # one epoch of its training: 200 samples in batches of 8
        {"name": "train-8", "kind": "train", "n": 8, "steps": 25},
        # the Table 2 analysis of a flow field
        {"name": "vortex-500x600-f64", "kind": "vortex", "nx": 500, "ny": 600, "dtype": "f64",
         "wall": "bounce-back"},
        # the Fig. 17 map: 153 probe series over 10,000 records
        {"name": "classify-153x10000", "kind": "classify", "series": 153, "samples": 10000},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: lattices from 48 to 4096 wide with aspect ratios 0.4 to
    2.0 and lattice Reynolds numbers the scheme is stable at, short calls and
    long ones, both storage types and wall schemes; batches, boxes, network
    batches, analysed fields and probe series of any size in use."""
    kind = rng.choice(["cavity", "cavity", "cavity", "nee", "batch", "box", "predict", "train",
                       "vortex", "classify"])
    dtype = rng.choice(["f64", "f32s"])
    if kind in ("cavity", "nee"):
        nx = _log(rng, 48, 4096 if kind == "cavity" else 1024)
        ny = max(32, min(4096, int(round(nx * rng.uniform(0.4, 2.0)))))
        # lattice Reynolds numbers of the paper's runs and below
        re = nx * rng.uniform(1.5, 12.0 if kind == "cavity" else 5.0)
        budget = 1.2e9 if dtype == "f32s" else 6e8
        steps = int(min(rng.choice([20, 100, 300, 1000]), max(20, budget / (nx * ny))))
        if steps > 20:
            steps = max(100, steps // 100 * 100)
        return {"kind": "cavity", "nx": nx, "ny": ny, "re": round(re, 1), "dtype": dtype,
                "wall": "bounce-back" if kind == "cavity" else "nee", "steps": steps}
    if kind == "batch":
        nx = _log(rng, 150, 500)
        n = rng.randint(4, 25)
        return {"kind": "batch", "nx": nx, "cavities": n, "re_lo": round(4.0 * nx, 1),
                "re_hi": round(rng.uniform(8.0, 14.0) * nx, 1), "dtype": dtype,
                "steps": rng.choice([500, 1000])}
    if kind == "box":
        sides = [_log(rng, 32, 192) for _ in range(3)]
        sites = sides[0] * sides[1] * sides[2]
        steps = int(max(100, min(rng.choice([100, 300, 500]), 2.0e9 / sites) // 100 * 100))
        return {"kind": "box", "nx": sides[0], "ny": sides[1], "nz": sides[2],
                "re": round(sides[0] * rng.uniform(1.0, 5.0), 1), "dtype": dtype,
                "steps": steps}
    if kind == "predict":
        return {"kind": "predict", "n": rng.randint(1, 16)}
    if kind == "train":
        return {"kind": "train", "n": rng.randint(2, 8), "steps": rng.randint(5, 25)}
    if kind == "vortex":
        nx = _log(rng, 64, 1024)
        ny = int(round(nx * rng.uniform(0.4, 2.0)))
        return {"kind": "vortex", "nx": nx, "ny": ny, "dtype": dtype,
                "wall": rng.choice(["bounce-back", "nee"])}
    return {"kind": "classify", "series": _log(rng, 1, 153), "samples": _log(rng, 300, 10000)}


# --------------------------------------------------------------------- inputs


def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _fields(nx, ny, seed, modes=6):
    """A smooth flow (rho, u_x, u_y), each [ny][nx] FP64 on the GPU: the
    velocity of a stream function of a few random cells that vanishes with its
    gradient at the walls, up to 0.04, and a density within 1e-3 of 1."""
    g = _generator(seed)
    x = (torch.arange(nx, device=DEV, dtype=torch.float64) + 0.5) / nx
    y = (torch.arange(ny, device=DEV, dtype=torch.float64) + 0.5) / ny
    a = torch.randn(modes, generator=g, device=DEV, dtype=torch.float64)
    ph = 2 * math.pi * torch.rand(4, modes, generator=g, device=DEV, dtype=torch.float64)
    k = torch.arange(1, modes + 1, device=DEV, dtype=torch.float64)
    sx, sy = torch.sin(math.pi * x) ** 2, torch.sin(math.pi * y) ** 2
    dsx = math.pi * torch.sin(2 * math.pi * x)
    dsy = math.pi * torch.sin(2 * math.pi * y)
    bx = torch.cos(math.pi * k[:, None] * x + ph[0][:, None])
    by = torch.cos(math.pi * k[:, None] * y + ph[1][:, None])
    dbx = -math.pi * k[:, None] * torch.sin(math.pi * k[:, None] * x + ph[0][:, None])
    dby = -math.pi * k[:, None] * torch.sin(math.pi * k[:, None] * y + ph[1][:, None])
    ux = (dsy * by + sy * dby).T @ (a[:, None] * (sx * bx)) / ny
    uy = -(sy * by).T @ (a[:, None] * (dsx * bx + sx * dbx)) / nx
    top = torch.maximum(ux.abs().max(), uy.abs().max())
    rho = torch.cos(2 * math.pi * y + ph[2, 0])[:, None] * torch.cos(2 * math.pi * x + ph[3, 0])
    return (1.0 + 1e-3 * rho).contiguous(), (ux * (0.04 / top)).contiguous(), \
        (uy * (0.04 / top)).contiguous()


def _sweep(case):
    """The batch's cavities (nx, ny, re): aspect ratios 0.4 ... 2.0 by Reynolds
    numbers between the case's two ends, five of each where there are 25."""
    n = case["cavities"]
    per = max(1, math.isqrt(n))
    ars = [0.4 + 1.6 * i / max(1, (n - 1) // per) for i in range((n + per - 1) // per)]
    res = [case["re_lo"] + (case["re_hi"] - case["re_lo"]) * i / max(1, per - 1)
           for i in range(per)]
    return [(case["nx"], int(round(case["nx"] * ar)), re) for ar in ars for re in res][:n]


def _populations3(case, seed):
    """A start for the box: f = w (1 + smooth random shift of 1 %), host FP64."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    rng = np.random.default_rng(seed)
    ax, ay, az = (np.sin(np.pi * (np.arange(m) + 0.5) / m) for m in (nx, ny, nz))
    shape = az[:, None, None] * ay[:, None] * ax
    f = np.empty((19, nz, ny, nx))
    for i in range(19):
        w = 1 / 3 if i == 0 else (1 / 18 if i < 7 else 1 / 36)
        np.multiply(shape, w * 0.01 * rng.uniform(-1, 1), out=f[i])
        f[i] += w
    return f


# (level, ci, co, real ci, real co) of the network's convolutions
_CONVS = ((0, 32, 32, 5, 32), (0, 32, 32, 32, 32), (1, 32, 64, 32, 64), (1, 64, 64, 64, 64),
          (2, 64, 128, 64, 128), (2, 128, 128, 128, 128), (3, 128, 256, 128, 256),
          (3, 256, 256, 256, 256), (2, 384, 128, 384, 128), (2, 128, 128, 128, 128),
          (1, 192, 64, 192, 64), (1, 64, 64, 64, 64), (0, 96, 32, 96, 32),
          (0, 32, 32, 32, 32), (0, 32, 32, 32, 3))
CANVAS_H, CANVAS_W = 256, 128


def _parameters(seed):
    """He-normal weights [9][ci][co] and small biases of every convolution,
    padding entries zero, in one FP32 array."""
    rng = np.random.default_rng(seed)
    parts = []
    for _, ci, co, cr, orl in _CONVS:
        w = np.zeros((9, ci, co), np.float32)
        w[:, :cr, :orl] = math.sqrt(2.0 / (9 * cr)) * rng.standard_normal((9, cr, orl),
                                                                       dtype=np.float32)
        b = np.zeros(co, np.float32)
        b[:orl] = 0.01 * rng.standard_normal(orl, dtype=np.float32)
        parts += [w.reshape(-1), b]
    return np.concatenate(parts)


def _samples(n, seed):
    rng = np.random.default_rng(seed + 1)
    return rng.uniform(100.0, 3000.0, n), rng.uniform(0.4, 2.0, n)


def _series(case, seed):
    """Probe series as a flow map records them: settled flows, oscillations
    with their harmonics, modulated and noisy ones, slow drifts."""
    rng = np.random.default_rng(seed)
    n, t = case["samples"], np.arange(case["samples"], dtype=np.float64)
    out = np.empty((case["series"], n))
    for s in range(case["series"]):
        kind = s % 5
        u0, amp = rng.uniform(-0.03, 0.03), rng.uniform(1e-3, 1e-2)
        period = rng.uniform(14.0, max(20.0, min(120.0, n / 12)))
        if kind == 0:       # settled
            out[s] = u0 + 1e-7 * np.exp(-t / n) * np.cos(2 * np.pi * t / period)
        elif kind == 1:     # periodic
            out[s] = u0 + amp * (np.cos(2 * np.pi * t / period + rng.uniform(0, 6))
                                 + 0.3 * np.cos(4 * np.pi * t / period + rng.uniform(0, 6)))
        elif kind == 2:     # two incommensurate oscillations
            out[s] = u0 + amp * (np.cos(2 * np.pi * t / period)
                                 + 0.8 * np.cos(2 * np.pi * t / (period * rng.uniform(1.3, 2.7))))
        elif kind == 3:     # chaotic: an oscillation with a wandering phase
            ph = np.cumsum(rng.normal(0.0, 0.25, n))
            out[s] = u0 + amp * np.cos(2 * np.pi * t / period + ph)
        else:               # a monotone approach
            out[s] = u0 + amp * np.exp(-t / (0.6 * n))
    return out


# -------------------------------------------------------------- prepare, run


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("cavity", "vortex"):
        nx, ny = case["nx"], case["ny"]
        c = lbm.Cavity(nx, ny, re=case.get("re", 4.0 * nx), u_lid=U_LID, dtype=case["dtype"],
                       wall=case["wall"])
        rho, ux, uy = _fields(nx, ny, seed)
        torch.cuda.synchronize()
        c.init_fields_device(rho, ux, uy)
        if kind == "vortex":
            return {"kind": kind, "c": c}
        return {"kind": kind, "c": c, "steps": case["steps"], "rho": rho, "ux": ux, "uy": uy}
    if kind == "batch":
        cav = _sweep(case)
        b = lbm.Batch([v[0] for v in cav], [v[1] for v in cav], [v[2] for v in cav],
                      u_lid=U_LID, dtype=case["dtype"])
        for k, (nx, ny, _) in enumerate(cav):
            f = _fields(nx, ny, seed + 100 * k)
            torch.cuda.synchronize()
            lbm.lbm_batch_init_fields_device(b.b, k, *f)
        n = len(cav)
        return {"kind": kind, "b": b, "n": n, "steps": case["steps"],
                "target": torch.empty((n, CANVAS_H, CANVAS_W, 3), device=DEV),
                "mask": torch.empty((n, CANVAS_H, CANVAS_W), device=DEV)}
    if kind == "box":
        c = lbm.Cube(case["nx"], case["ny"], case["nz"], re=case["re"], u_lid=U_LID,
                     dtype=case["dtype"])
        c.set_populations(_populations3(case, seed))
        return {"kind": kind, "c": c, "steps": case["steps"]}
    if kind in ("predict", "train"):
        n = case["n"]
        s = lbm.Surrogate(n)
        s.set_params(_parameters(seed))
        re, ar = _samples(n, seed)
        st = {"kind": kind, "s": s, "re": re, "ar": ar}
        if kind == "predict":
            st["out"] = torch.empty((n, CANVAS_H, CANVAS_W, 3), device=DEV)
            return st
        target = torch.zeros((n, CANVAS_H, CANVAS_W, 3), device=DEV)
        mask = torch.zeros((n, CANVAS_H, CANVAS_W), device=DEV)
        for i in range(n):
            rows = int(np.rint(128.0 * ar[i]))
            rho, ux, uy = _fields(CANVAS_W, rows, seed + 10 * i)
            target[i, :rows] = torch.stack([100.0 * (rho - 1.0), ux / U_LID, uy / U_LID],
                                           dim=-1).float()
            mask[i, :rows] = 1.0
        return {**st, "target": target, "mask": mask, "steps": case["steps"]}
    if kind == "classify":
        return {"kind": kind, "series": torch.from_numpy(_series(case, seed)).to(DEV)}
    raise ValueError(kind)


_VORTEX_FLOOR = 1e-3      # of Psi, lattice units
_STATES = {v: k for k, v in lbm.FLOW_STATES.items()}
_RECORD = ("period", "amplitude", "mean", "std", "mismatch", "cycle", "cycle_mismatch")


def run(state):
    kind = state["kind"]
    if kind == "cavity":
        c = state["c"]
        c.step(state["steps"])
        c.moments_device(state["rho"], state["ux"], state["uy"])
        out = {"rho": state["rho"], "ux": state["ux"], "uy": state["uy"]}
        if state["steps"] % 100 == 0:
            out["residual"] = c.residual()[0]
        return out
    if kind == "batch":
        b = state["b"]
        b.step(state["steps"])
        for k in range(state["n"]):
            b.canvas(k, state["target"][k], state["mask"][k])
        return {"target": state["target"], "mask": state["mask"], "residuals": b.residuals()}
    if kind == "box":
        c = state["c"]
        c.step(state["steps"])
        rho, ux, uy, uz = c.moments()
        return {"rho": rho, "ux": ux, "uy": uy, "uz": uz, "residual": c.residual()[0]}
    if kind == "predict":
        state["s"].forward(state["re"], state["ar"], state["out"])
        return {"out": state["out"]}
    if kind == "train":
        loss = 0.0
        for _ in range(state["steps"]):
            loss = state["s"].train_step(state["re"], state["ar"], state["target"],
                                         state["mask"], 1e-3)
        params, grads = state["s"].get_params(with_grads=True)
        return {"loss": loss, "params": params, "grads": grads}
    if kind == "vortex":
        c = state["c"]
        ext = c.vortex_extrema()
        table = np.zeros((64, 6))        # the centres, one row each
        centres, count = c.vortex_centres(_VORTEX_FLOOR)
        bottom = c.bottom_vortex_count(_VORTEX_FLOOR)
        psi = c.stream_function()
        for row, v in zip(table, centres):
            row[:] = v.psi, v.x, v.y, v.ix, v.iy, v.kind
        return {"psi": psi,
                "extrema": np.array([[v.psi, v.x, v.y] for v in ext]),
                "extrema_site": np.array([[v.ix, v.iy, v.kind] for v in ext]),
                "centres": table[:, :3].copy(),
                "centres_site": table[:, 3:].astype(np.int64),
                "counts": np.array([count, bottom])}
    recs = lbm.lbm_classify_series(state["series"], 1e-4 * U_LID, 0.05)
    return {"values": np.array([[r[k] for k in _RECORD] for r in recs]),
            "states": np.array([[_STATES[r["state"]], r["lag"]] for r in recs])}


# ----------------------------------------------------------------------- work


def work(case):
    kind = case["kind"]
    if kind in ("cavity", "batch"):
        esz = 8 if case["dtype"] == "f64" else 4
        cav = _sweep(case) if kind == "batch" else [(case["nx"], case["ny"], 0.0)]
        sites = sum(c[0] * c[1] for c in cav)
        out = 16.0 * CANVAS_H * CANVAS_W * len(cav) if kind == "batch" else 24.0 * sites
        # a state read once and written once; about 120 operations an update
        return {"bytes": sites * 2.0 * 9 * esz + out, "flops": 120.0 * sites * case["steps"]}
    if kind == "box":
        esz = 8 if case["dtype"] == "f64" else 4
        sites = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": sites * (2.0 * 19 * esz + 32.0), "flops": 240.0 * sites * case["steps"]}
    if kind in ("predict", "train"):
        fl = [2.0 * 9 * cr * orl * (CANVAS_H >> l) * (CANVAS_W >> l)
              for l, _, _, cr, orl in _CONVS]
        params = sum(9 * ci * co + co for _, ci, co, _, _ in _CONVS)
        n, pix = case["n"], CANVAS_H * CANVAS_W
        if kind == "predict":
            return {"bytes": 2.0 * params + 12.0 * n * pix, "flops": n * sum(fl)}
        return {"bytes": case["steps"] * (28.0 * params + 16.0 * n * pix),
                "flops": case["steps"] * n * (2 * sum(fl) + sum(fl[1:]))}
    if kind == "vortex":
        esz = 8 if case["dtype"] == "f64" else 4
        sites = case["nx"] * case["ny"]
        return {"bytes": sites * (9.0 * esz + 8.0), "flops": 40.0 * sites}
    n, s = case["samples"], case["series"]
    lags = n // 3
    return {"bytes": 8.0 * n * s + 72.0 * s, "flops": 3.0 * s * lags * (n - 0.5 * lags)}


# ---------------------------------------------------------------------- exact

_C2 = ((0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1))
_W2 = (4 / 9,) + (1 / 9,) * 4 + (1 / 36,) * 4
_OPP2 = (0, 3, 4, 1, 2, 7, 8, 5, 6)
_C3 = ((0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
       (1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1),
       (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1))


def _slices(c, n):
    """(destination, source) of a shift by c along an axis of n sites."""
    return (slice(max(c, 0), n + min(c, 0)), slice(max(-c, 0), n - max(c, 0)))


def _moments2(f):
    rho = f.sum(0)
    ux = (f[1] - f[3] + f[5] - f[6] + f[8] - f[7]) / rho
    uy = (f[2] - f[4] + f[5] + f[6] - f[7] - f[8]) / rho
    return rho, ux, uy


def _equilibrium2(rho, ux, uy):
    usq = 1.5 * (ux * ux + uy * uy)
    return torch.stack([w * rho * (1.0 + 3.0 * (cx * ux + cy * uy)
                                   + 4.5 * (cx * ux + cy * uy) ** 2 - usq)
                        for (cx, cy), w in zip(_C2, _W2)])


def _stream2(f):
    """Populations of a stack [9][..., ny, nx] after streaming; half-way
    bounce-back where a link comes through a wall, the lid at the top."""
    ny, nx = f.shape[-2:]
    g = torch.empty_like(f)
    for i, (cx, cy) in enumerate(_C2):
        g[i] = f[_OPP2[i]]
        (dx, sx), (dy, sy) = _slices(cx, nx), _slices(cy, ny)
        if cy < 0 and cx:
            g[i, ..., ny - 1, :] += cx * U_LID / 6.0
        g[i][..., dy, dx] = f[i][..., sy, sx]
    return g


def _evolve2(rho, ux, uy, omega, steps, wall):
    """(moments, velocity 100 steps before) after `steps` steps of the lattice
    BGK update from equilibrium; fields [..., ny, nx]."""
    f = _equilibrium2(rho, ux, uy)
    before = None
    ny, nx = rho.shape[-2:]
    if wall == "nee":
        ry = torch.arange(ny, device=rho.device).clamp(1, ny - 2)
        rx = torch.arange(nx, device=rho.device).clamp(1, nx - 2)
        on_wall = torch.ones((ny, nx), dtype=torch.bool, device=rho.device)
        on_wall[1:-1, 1:-1] = False
        uw = torch.zeros((ny, nx), dtype=torch.float64, device=rho.device)
        uw[-1] = U_LID
        zero = torch.zeros_like(uw)
    for t in range(steps):
        if t == steps - 100:
            before = _moments2(f)[1:]
        if wall == "nee":
            g = torch.empty_like(f)
            for i, (cx, cy) in enumerate(_C2):
                g[i, 1:-1, 1:-1] = f[i, 1 - cy:ny - 1 - cy, 1 - cx:nx - 1 - cx]
            g = g[:, ry][:, :, rx]
            r, u, v = _moments2(g)
            eq = _equilibrium2(r, u, v)
            part = (1.0 - omega) * (g - eq)
            f = torch.where(on_wall, _equilibrium2(r, uw, zero), eq) + part
        else:
            g = _stream2(f)
            eq = _equilibrium2(*_moments2(g))
            f = g + omega * (eq - g)
    return _moments2(f), before


def _residual(u, before):
    num = sum(((a - b) ** 2).sum((-2, -1)) for a, b in zip(u, before))
    return torch.sqrt(num / sum((b ** 2).sum((-2, -1)) for b in before))


def _exact_cavity(case, seed):
    nx, ny = case["nx"], case["ny"]
    rho, ux, uy = _fields(nx, ny, seed)
    rho = rho * (nx * ny / rho.sum())
    width = nx - 1 if case["wall"] == "nee" else nx
    omega = 1.0 / (3.0 * U_LID * width / case["re"] + 0.5)
    (rho, ux, uy), before = _evolve2(rho, ux, uy, omega, case["steps"], case["wall"])
    out = {"rho": rho, "ux": ux, "uy": uy}
    if case["steps"] % 100 == 0:
        out["residual"] = float(_residual((ux, uy), before))
    return out


def _bilinear(field, rows, nx):
    """Values of [ny][nx] site-centred fields at the canvas pixels' centres."""
    ny = field.shape[-2]

    def place(m, n):
        p = ((torch.arange(m, device=DEV, dtype=torch.float64) + 0.5) / 128.0 * nx - 0.5)
        p = p.clamp(0.0, n - 1.0)
        i = p.floor().clamp(max=n - 2).long()
        return i, p - i
    (j, ty), (i, tx) = place(rows, ny), place(CANVAS_W, nx)
    ty = ty[:, None]
    a, b = field[j][:, i], field[j][:, i + 1]
    c, d = field[j + 1][:, i], field[j + 1][:, i + 1]
    return (1 - ty) * ((1 - tx) * a + tx * b) + ty * ((1 - tx) * c + tx * d)


def _exact_batch(case, seed):
    cav = _sweep(case)
    if sum(c[0] * c[1] for c in cav) * case["steps"] > 8e9:
        return None
    target = torch.zeros((len(cav), CANVAS_H, CANVAS_W, 3), device=DEV, dtype=torch.float64)
    mask = torch.zeros((len(cav), CANVAS_H, CANVAS_W), device=DEV, dtype=torch.float64)
    res = np.empty(len(cav))
    for nx, ny in sorted({c[:2] for c in cav}):      # equal lattices side by side
        ks = [k for k, c in enumerate(cav) if c[:2] == (nx, ny)]
        fl = [_fields(nx, ny, seed + 100 * k) for k in ks]
        rho, ux, uy = (torch.stack([f[q] for f in fl]) for q in range(3))
        rho = rho * (nx * ny / rho.sum((-2, -1), keepdim=True))
        omega = torch.tensor([1.0 / (3.0 * U_LID * nx / cav[k][2] + 0.5) for k in ks],
                             device=DEV, dtype=torch.float64)[:, None, None]
        (rho, ux, uy), before = _evolve2(rho, ux, uy, omega, case["steps"], "bounce-back")
        res[ks] = _residual((ux, uy), before).cpu().numpy()
        rows = int(np.rint(128.0 * ny / nx))
        for q, k in enumerate(ks):
            target[k, :rows, :, 0] = 100.0 * (_bilinear(rho[q], rows, nx) - 1.0)
            target[k, :rows, :, 1] = _bilinear(ux[q], rows, nx) / U_LID
            target[k, :rows, :, 2] = _bilinear(uy[q], rows, nx) / U_LID
            mask[k, :rows] = 1.0
    return {"target": target, "mask": mask, "residuals": res}


def _exact_box(case, seed):
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if nx * ny * nz * case["steps"] > 2.5e9:
        return None
    f = torch.from_numpy(_populations3(case, seed)).to(DEV)
    omega = 1.0 / (3.0 * U_LID * nx / case["re"] + 0.5)
    w = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
    before = None

    def moments(f):
        rho = f.sum(0)
        return rho, *(sum(c[a] * f[i] for i, c in enumerate(_C3) if c[a]) / rho
                      for a in range(3))

    def collide(f):
        rho, ux, uy, uz = moments(f)
        usq = 1.5 * (ux * ux + uy * uy + uz * uz)
        for i, (a, b, c) in enumerate(_C3):
            cu = a * ux + b * uy + c * uz
            f[i] += omega * (w[i] * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - usq) - f[i])
        return f

    f = collide(f)
    g = torch.empty_like(f)
    for t in range(case["steps"]):
        if t == case["steps"] - 100:
            before = moments(f)[1:]
        for i, (a, b, c) in enumerate(_C3):
            o = i if i == 0 else (i + 1 if i % 2 else i - 1)
            g[i] = f[o]
            if b < 0 and a:
                g[i, :, ny - 1] += a * U_LID / 6.0
            (dx, sx), (dy, sy), (dz, sz) = _slices(a, nx), _slices(b, ny), _slices(c, nz)
            g[i][dz, dy, dx] = f[i][sz, sy, sx]
        f, g = collide(g), f
    rho, ux, uy, uz = moments(f)
    num = sum(((p - q) ** 2).sum() for p, q in zip((ux, uy, uz), before))
    res = float(torch.sqrt(num / sum((q ** 2).sum() for q in before)))
    return {"rho": rho, "ux": ux, "uy": uy, "uz": uz, "residual": res}


def _exact_predict(case, seed):
    """The U-Net in 64 bits: 3 x 3 convolutions as nine shifted products."""
    n = case["n"]
    p = torch.from_numpy(_parameters(seed)).to(DEV).double()
    re, ar = _samples(n, seed)
    x = torch.zeros((n, CANVAS_H, CANVAS_W, 32), device=DEV, dtype=torch.float64)
    px = (torch.arange(CANVAS_W, device=DEV, dtype=torch.float64) + 0.5) / 128.0
    py = (torch.arange(CANVAS_H, device=DEV, dtype=torch.float64) + 0.5) / 128.0
    for i in range(n):
        x[i, :int(np.rint(128.0 * ar[i])), :, 0] = 1.0
        x[i, :, :, 1] = px
        x[i, :, :, 2] = py[:, None]
        x[i, :, :, 3] = re[i] / 3000.0
        x[i, :, :, 4] = ar[i] / 2.0
    at = [0]

    def conv(x, k, relu=True):
        _, ci, co, _, _ = _CONVS[k]
        wt = p[at[0]:at[0] + 9 * ci * co].reshape(9, ci, co)
        bias = p[at[0] + 9 * ci * co:at[0] + 9 * ci * co + co]
        at[0] += 9 * ci * co + co
        h, wd = x.shape[1:3]
        pad = torch.zeros((n, h + 2, wd + 2, ci), device=DEV, dtype=torch.float64)
        pad[:, 1:-1, 1:-1] = x
        y = bias.expand(n * h * wd, co).clone()
        for t in range(9):
            part = pad[:, t // 3:t // 3 + h, t % 3:t % 3 + wd].reshape(-1, ci)
            y += part @ wt[t]
        y = y.reshape(n, h, wd, co)
        return y.clamp(min=0.0) if relu else y

    def pool(x):
        return 0.25 * (x[:, ::2, ::2] + x[:, 1::2, ::2] + x[:, ::2, 1::2] + x[:, 1::2, 1::2])

    def up(x):
        return x.repeat_interleave(2, 1).repeat_interleave(2, 2)

    skips = []
    for level in range(3):
        x = conv(conv(x, 2 * level), 2 * level + 1)
        skips.append(x)
        x = pool(x)
    x = conv(conv(x, 6), 7)
    for k in (8, 10, 12):
        x = conv(conv(torch.cat([up(x), skips.pop()], dim=-1), k), k + 1)
    return {"out": conv(x, 14, relu=False)[..., :3].contiguous()}


def _exact_vortex(case, seed):
    """Psi alone: up each column from the bottom wall, the midpoint rule on
    site centres or the trapezoid rule on nodes."""
    _, ux, _ = _fields(case["nx"], case["ny"], seed)
    up = torch.cumsum(ux, 0)
    if case["wall"] == "nee":
        psi = -(up - 0.5 * ux - 0.5 * ux[0])
    else:
        psi = -(up - 0.5 * ux)
    return {"psi": psi.contiguous()}


def _exact_classify(case, seed):
    n, s = case["samples"], case["series"]
    host = _series(case, seed)
    u = torch.from_numpy(host).to(DEV)
    lags = n // 3
    d = torch.empty((lags, s), device=DEV, dtype=torch.float64)
    for t in range(1, lags + 1):
        d[t - 1] = (u[:, t:] - u[:, :-t]).square().mean(1)
    d = (d / u.var(1, unbiased=False)).cpu().numpy()
    out = np.zeros((s, len(_RECORD)))
    for q in range(s):
        mean, std = host[q].mean(), host[q].std()
        amp = host[q].max() - host[q].min()
        period = mis = cyc = cyc_mis = 0.0
        if amp > 1e-4 * U_LID:
            a, b, c = d[:-2, q], d[1:-1, q], d[2:, q]
            seen = np.logical_or.accumulate(a > 1.0)
            best, found = np.inf, False
            for j in np.nonzero(seen & (a > b) & (b <= c))[0]:
                curv = a[j] - 2 * b[j] + c[j]
                at, vertex = float(j + 2), b[j]
                if curv > 0:
                    at += 0.5 * (a[j] - c[j]) / curv
                    vertex -= (a[j] - c[j]) ** 2 / (8 * curv)
                m = math.sqrt(max(vertex, 0.0))
                if best == np.inf:
                    cyc, cyc_mis = at, m
                best = min(best, m)
                if m <= 0.05:
                    period, mis, found = at, m, True
                    break
            if not found:
                mis = best
                if best == np.inf:
                    cyc_mis = np.inf
        out[q] = period, amp, mean, std, mis, cyc, cyc_mis
    return {"values": out}


def exact(case, seed):
    kind = case["kind"]
    if kind == "cavity":
        return _exact_cavity(case, seed)
    if kind == "batch":
        return _exact_batch(case, seed)
    if kind == "box":
        return _exact_box(case, seed)
    if kind == "predict":
        return _exact_predict(case, seed)
    if kind == "vortex":
        return _exact_vortex(case, seed)
    if kind == "classify":
        return _exact_classify(case, seed)
    return None          # training: 25 steps in bf16 have no 64-bit counterpart
