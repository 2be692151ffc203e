"""The measured work of this framework: its calls over the sizes they are used at.

A case is a plain dict; prepare() makes what a user's program holds before the call (device
inputs from the seed alone, the simulation, context or network handle), run() is one pass
through the public entry points, exact() the same outputs from plain numpy / torch in 64
bits.  Kinds:

  loop      two steps of the box geometries' loop, replayed from a HIP graph (the form the
            loop is run in for thousands of steps), with the time averages sampled
  cylinder  one step of the open cylinder's loop, on its adaptive quadtree or (levels 0)
            on the uniform grid, with injection and deletion, launched eagerly
  resort    the loop's re-sort alone: particles grouped by their previous cell, sorted by
            their new one, with the moment records and the time-average sums
  closure   the exact 9x9 closure of a batch of cells
  nn        the 27-feature learned closure of a batch of cells (checked or not)
  lite      the 16-input learned closure on third-order records (unchecked)
  train     one Adam step of either network on a batch (mean squared error, or the closure
            residual of the 27-feature network's fine-tuning)
  grad      particle velocities -> coefficients and back (reverse mode)
"""
import math

import numpy as np
import torch

from paper_2606_15622_amd import fpgpu as F
from paper_2606_15622_amd import inputs as I
from paper_2606_15622_amd.autograd import ExactClosure

EPS_HAT = 0.01
LR = 1e-4
KN = 0.5


def listed():
    return [
        # the smallest use: the 1-D channel of the training data (100 cells x 100 particles in
        # FP64), thousands of steps, bound by launches and latency
        {"name": "couette_1e4_f64", "kind": "loop", "geometry": "couette1d", "cells": 100, "ppc": 100,
         "precision": "f64", "conserve": "exact", "sample": True},
        # the headline: the lid-driven cavity of the published runs, FP32 particles
        {"name": "cavity_1e6_f32", "kind": "loop", "geometry": "cavity2d", "cells": 100, "ppc": 100,
         "precision": "f32", "conserve": "exact", "sample": True},
        # the largest: a cavity beyond the last-level cache
        {"name": "cavity_2e7_f32", "kind": "loop", "geometry": "cavity2d", "cells": 448, "ppc": 100,
         "precision": "f32", "conserve": "exact", "sample": True},
        # Mach 10 flow past the cylinder on the adaptive quadtree, uneven leaves of few particles
        {"name": "cylinder_tree_1.8e7", "kind": "cylinder", "levels": 2, "nx": 400, "ny": 300,
         "particles": 18000000, "sample": True},
        # the re-sort by itself on an odd grid with few particles per cell, FP64 storage
        {"name": "resort_ragged_f64", "kind": "resort", "cells": 211, "ppc": 33, "precision": "f64"},
        # the closures on a batch of cells (the closure comparison of the benchmark)
        {"name": "closure_1e6", "kind": "closure", "cells": 1000000},
        {"name": "nn_checked_1e6", "kind": "nn", "cells": 1000000, "checked": True, "relax": 1.0},
        {"name": "lite_1e6", "kind": "lite", "cells": 1000003, "relax": 1.0},
        # training at the default batch, once per step over some 1e4 steps
        {"name": "train_nn_4096", "kind": "train", "net": "nn", "loss": "mse", "batch": 4096},
        {"name": "train_lite_4096", "kind": "train", "net": "lite", "loss": "mse", "batch": 4096},
        # fine-tuning on the closure residual at its default batch
        {"name": "finetune_nn_2e5", "kind": "train", "net": "nn", "loss": "residual", "batch": 200000},
        # differentiation: 1e4 cells of 10 to 500 particles
        {"name": "grad_1e4_cells_f64", "kind": "grad", "cells": 10000, "lo": 10, "hi": 500, "precision": "f64"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["loop", "loop", "cylinder", "resort", "closure", "nn", "lite", "train", "train", "grad"])
    if kind == "loop":
        n, ppc = _log(rng, 1e4, 1e7), _log(rng, 20, 200)
        geo = rng.choice(["couette1d", "cavity2d", "cavity2d"])
        cells = max(10, n // ppc) if geo == "couette1d" else max(8, int(math.sqrt(n / ppc)))
        return {"kind": kind, "geometry": geo, "cells": cells, "ppc": ppc, "precision": rng.choice(["f32", "f32", "f64"]),
                "conserve": rng.choice(["exact", "exact", "paper"]), "sample": rng.random() < 0.7}
    if kind == "cylinder":
        q = _log(rng, 12, 100)   # the box is 4 : 3
        return {"kind": kind, "levels": rng.choice([0, 1, 2]), "nx": 4 * q, "ny": 3 * q,
                "particles": min(10000000, 12 * q * q * _log(rng, 30, 200)), "sample": rng.random() < 0.7}
    if kind == "resort":
        n, ppc = _log(rng, 1e4, 1e7), _log(rng, 20, 200)
        return {"kind": kind, "cells": max(8, int(math.sqrt(n / ppc))), "ppc": ppc, "precision": rng.choice(["f32", "f64"])}
    if kind == "closure":
        return {"kind": kind, "cells": _log(rng, 1e3, 2e6)}
    if kind == "nn":
        return {"kind": kind, "cells": _log(rng, 1e3, 1e6), "checked": rng.random() < 0.5, "relax": rng.choice([1.0, 0.2])}
    if kind == "lite":
        return {"kind": kind, "cells": _log(rng, 1e3, 1e6), "relax": rng.choice([1.0, 0.2])}
    if kind == "train":
        net = rng.choice(["nn", "lite"])
        loss = "mse" if net == "lite" else rng.choice(["mse", "residual"])
        return {"kind": kind, "net": net, "loss": loss, "batch": _log(rng, 500, 100000 if net == "lite" else 200000)}
    lo = _log(rng, 5, 50)
    return {"kind": kind, "cells": _log(rng, 300, 20000), "lo": lo, "hi": lo * rng.randint(2, 10), "precision": rng.choice(["f32", "f64"])}


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, int(seed))


def run(state):
    return _RUN[state["kind"]](state)


def exact(case, seed):
    fn = _EXACT.get(case["kind"])
    return fn(case, int(seed)) if fn else None


def work(case):
    k = case["kind"]
    if k == "loop":
        # state read and written once per step, the sums of every cell read and written
        two_d = case["geometry"] != "couette1d"
        nc = case["cells"] ** 2 if two_d else case["cells"]
        n, w = nc * case["ppc"], 4 if case["precision"] == "f32" else 8
        return {"bytes": 2.0 * (2 * n * ((5 if two_d else 4) * w + 4) + nc * (224 if case["sample"] else 0)),
                "flops": 2.0 * (250 * n + 1000 * nc)}
    if k == "cylinder":
        n = case["particles"]
        return {"bytes": 48.0 * n, "flops": 250.0 * n}
    if k == "resort":
        nc, w = case["cells"] ** 2, 4 if case["precision"] == "f32" else 8
        n = nc * case["ppc"]
        return {"bytes": n * (2.0 * (5 * w + 8) + 4) + nc * (8 + 256 + 224.0), "flops": 60.0 * n}
    n = case.get("cells", 0)
    if k == "closure":
        return {"bytes": 388.0 * n, "flops": 900.0 * n}
    if k == "nn":
        return {"bytes": 388.0 * n, "flops": (77824.0 + (500 if case["checked"] else 0)) * n}
    if k == "lite":
        return {"bytes": (168 + 132.0) * n, "flops": 2.0 * 204041 * n}
    if k == "train":
        B = case["batch"]
        p, row = (38537, 27 * 4 + (36 if case["loss"] == "mse" else 720)) if case["net"] == "nn" else (204041, 100)
        return {"bytes": float(B * row + 24 * p), "flops": 6.0 * p * B}
    n = case["cells"] * (case["lo"] + case["hi"]) / 2
    w = 4 if case["precision"] == "f32" else 8
    return {"bytes": 6.0 * w * n, "flops": 250.0 * n + 2500.0 * case["cells"]}


# ---- inputs -----------------------------------------------------------------------------
def _gen(seed, device="cuda"):
    return torch.Generator(device=device).manual_seed(seed)


def _rand(g, *shape, dtype=torch.float64):
    return torch.rand(*shape, generator=g, device=g.device, dtype=dtype)


def _randn(g, *shape, dtype=torch.float64):
    return torch.randn(*shape, generator=g, device=g.device, dtype=dtype)


def _box(case, seed):
    if case["geometry"] == "couette1d":
        return I.couette(kn=0.1, ncell=case["cells"], ppc=case["ppc"], precision=case["precision"],
                         conserve=case["conserve"], seed=seed)
    return I.cavity(kn=1.0, ncell=case["cells"], ppc=case["ppc"], precision=case["precision"],
                    conserve=case["conserve"], seed=seed)


def _box_state(w, seed):
    """ppc particles in every cell, uniform inside it, Maxwellian at the initial temperature."""
    g = _gen(seed)
    nx, ny, ppc = int(w["nx"]), int(w["ny"]), int(w["ppc"])
    n = nx * ny * ppc
    dt = torch.float32 if w["precision"] == "f32" else torch.float64
    cell = torch.arange(nx * ny, device="cuda").repeat_interleave(ppc)
    x = (w["x0"] + (cell % nx + _rand(g, n)) * w["dx"]).to(dt)
    y = (w["y0"] + (cell // nx + _rand(g, n)) * w["dy"]).to(dt) if w["geometry"] != "couette1d" else torch.zeros(n, dtype=dt)
    s = math.sqrt(w["R"] * w["T_init"])
    st = {"x": x, "y": y}
    for k in ("vx", "vy", "vz"):
        st[k] = (_randn(g, n) * s).to(dt)
    st = {k: v.cpu().numpy() for k, v in st.items()}
    st["pid"] = np.arange(n, dtype=np.uint32)
    return st


def _prep_loop(case, seed):
    w = _box(case, seed)
    sim = F.GraphSimulation(w, _box_state(w, seed), step0=1)
    sim.step(0, sample=case["sample"])        # the first sort of a run is the general one
    sim.run_pairs(0, sample=case["sample"])   # captures the two steps
    return {"kind": "loop", "sim": sim, "sample": case["sample"]}


def _run_loop(s):
    sim = s["sim"]
    sim.run_pairs(1, sample=s["sample"])
    a = sim.a
    out = {"x": a.x, "vx": a.vx, "vy": a.vy, "vz": a.vz, "pid": a.pid, "key": a.key, "offsets": sim.offsets,
           "mom": sim.mom, "rec": sim.rec, "status": sim.status, "samp": sim.samp}
    if a.two_d:
        out["y"] = a.y
    return out


def _shock_sums(w, xc, yc, size):
    """Sums of one sampled step for cells centred at xc, yc: a detached bow shock's compressed
    and heated layer in front of and beside the cylinder, free stream elsewhere."""
    r = np.hypot(xc, yc)
    front = -0.13 + 1.8 * yc * yc          # the shock's parabola, ahead of the body
    layer = (xc > front) & (xc < 0.12 + 0.5 * np.abs(yc)) & (r > 0.08)
    rho = np.where(layer, 4.0, 1.0)
    T = np.where(layer, 8.0, 1.0) * w["T_inf"]
    acc = np.zeros((xc.shape[0], 16))
    n = rho * w["n_inf"] * size * size * w["depth"] / w["fnum"]
    acc[:, 0], acc[:, 13] = n, 1.0
    acc[:, 1] = n * w["u_inf"][0]
    th = w["R"] * T
    acc[:, 4], acc[:, 7], acc[:, 9] = n * (th + w["u_inf"][0] ** 2), n * th, n * th
    return acc


def _prep_cylinder(case, seed):
    L = case["levels"]
    nx, ny = case["nx"] << L, case["ny"] << L
    cell = 0.8 / nx
    area = 0.8 * 0.6 - math.pi * 0.01
    fnum = 1e20 * area / case["particles"]
    w = I.cylinder(cell=cell, nx=nx, ny=ny, fnum=fnum, precision="f32", seed=seed)
    g = _gen(seed)
    n = case["particles"]
    # free stream in the gas part of the box: draws that fall inside the body are left out
    xy = _rand(g, int(n * 1.08) + 1000, 2)
    x, y = w["x0"] + xy[:, 0] * w["lx"], w["y0"] + xy[:, 1] * w["ly"]
    out = torch.nonzero(x * x + y * y > 0.01)[:n, 0]
    s = math.sqrt(w["R"] * w["T_inf"])
    st = {"x": x[out].float(), "y": y[out].float()}
    n = int(out.shape[0])
    for k, u in zip(("vx", "vy", "vz"), w["u_inf"]):
        st[k] = (_randn(g, n) * s + u).float()
    st = {k: v.cpu().numpy() for k, v in st.items()}
    st["pid"] = np.arange(n, dtype=np.uint32)
    if L == 0:
        sim = F.OpenSimulation(w, st)
    else:
        base = w["n_inf"] * (cell * (1 << L)) ** 2 * w["depth"] / w["fnum"]
        prm = dict(tau_grad=0.10, tau_coarse=0.05, shock_factor=1.2, p_inf=w["n_inf"] * I.KB * w["T_inf"],
                   n_max=1e30, n_grad=0.2 * base, eps=1e-300, age_min=2000)
        sim = F.AMRSimulation(w, st, L, prm, 0)
        for _ in range(L):
            lm = sim.tree()[2].reshape(ny, nx)
            fy, fx = np.divmod(np.arange(nx * ny), nx)
            cnt = np.bincount(lm.ravel(), minlength=sim.ncell)
            xc = w["x0"] + (np.bincount(lm.ravel(), fx + 0.5, sim.ncell) / cnt) * cell
            yc = w["y0"] + (np.bincount(lm.ravel(), fy + 0.5, sim.ncell) / cnt) * cell
            sim.acc[:sim.ncell] = torch.from_numpy(_shock_sums(w, xc, yc, cell * np.sqrt(cnt))).cuda()
            sim.adapt(1)
    sim.step(0, sample=case["sample"])
    return {"kind": "cylinder", "sim": sim, "step": 1, "sample": case["sample"]}


def _run_cylinder(s):
    sim = s["sim"]
    sim.step(s["step"], sample=s["sample"])
    s["step"] += 1
    a, nc = sim.a, sim.ctx.ncell
    return {"x": a.x, "y": a.y, "vx": a.vx, "vy": a.vy, "vz": a.vz, "pid": a.pid, "key": a.key, "n": a.n_dev,
            "offsets": sim.offsets, "mom": sim.mom[:nc], "rec": sim.rec[:nc], "status": sim.status[:nc],
            "samp": sim.samp[:nc]}


def _resort_state(case, seed):
    """A sorted cavity after one flight: grouped by the old cell, keyed by the new one."""
    w = I.cavity(kn=1.0, ncell=case["cells"], ppc=case["ppc"], precision=case["precision"], seed=seed)
    st = _box_state(w, seed)
    old = np.repeat(np.arange(w["nx"] * w["ny"]), w["ppc"])
    rng = np.random.default_rng(seed)
    for k, v in (("x", "vx"), ("y", "vy")):
        p = st[k] + st[v] * w["dt"]
        L = w["lx"]
        st[k] = np.clip(np.where(p < 0, -p, np.where(p > L, 2 * L - p, p)), 0.0, L).astype(st[k].dtype)
    kx = np.clip(np.floor(st["x"].astype(np.float64) / w["dx"]), 0, w["nx"] - 1).astype(np.int64)
    ky = np.clip(np.floor(st["y"].astype(np.float64) / w["dy"]), 0, w["ny"] - 1).astype(np.int64)
    st["key"] = (ky * w["nx"] + kx).astype(np.int32)
    st["pid"] = rng.permutation(old.shape[0]).astype(np.uint32)
    off = np.arange(w["nx"] * w["ny"] + 1, dtype=np.int32) * np.int32(w["ppc"])
    return w, st, off


def _prep_resort(case, seed):
    w, st, off = _resort_state(case, seed)
    n, nc = st["x"].shape[0], off.shape[0] - 1
    ctx = F.Context(w, n)
    src = F.Particles.from_numpy(w, st)
    dst = F.Particles(n, src.dtype, True)
    f64 = dict(dtype=torch.float64, device="cuda")
    return {"kind": "resort", "ctx": ctx, "src": src, "dst": dst, "off0": torch.from_numpy(off).cuda(),
            "off": torch.zeros(nc + 1, dtype=torch.int32, device="cuda"),
            "perm": torch.zeros(n, dtype=torch.int32, device="cuda"),
            "mom": torch.zeros((nc, 32), **f64), "samp": torch.zeros((nc, 16), **f64)}


def _run_resort(s):
    s["ctx"].rebin(s["src"], s["off0"], s["dst"], s["off"], s["perm"], s["mom"], s["samp"])
    d = s["dst"]
    return {"x": d.x, "y": d.y, "vx": d.vx, "vy": d.vy, "vz": d.vz, "pid": d.pid, "key": d.key,
            "offsets": s["off"], "perm": s["perm"], "mom": s["mom"], "samp": s["samp"]}


# ---- moment records of cells ---------------------------------------------------------------
def _monomials(c):
    """[n][m][3] central velocities -> the 26 monomials of the record, in its order."""
    a, b, d = c[..., 0], c[..., 1], c[..., 2]
    c2 = a * a + b * b + d * d
    P = [a * a, a * b, a * d, b * b, b * d, d * d]
    T = [a * a * a, a * a * b, a * a * d, a * b * b, a * b * d, a * d * d, b * b * b, b * b * d, b * d * d, d * d * d]
    return P + T + [p * c2 for p in P] + [q * c2 * c2 for q in (a, b, d)] + [c2 ** 3]


def _records(n, seed, low=False):
    """Moment records of n cells of about 100 particles drawn from skewed anisotropic
    Gaussians (stress, heat flux and the higher moments non-zero); low: third order only."""
    g = _gen(seed)
    out = torch.zeros((n, 32), dtype=torch.float64, device="cuda")
    m, step = 160, 32768
    for i in range(0, n, step):
        k = min(step, n - i)
        cnt = torch.poisson(torch.full((k,), 100.0, device="cuda"), generator=g).clamp(1, m).double()
        th = I.KB / I.MASS_AR * (250.0 + 150.0 * _rand(g, k, 1, 1))
        z = _randn(g, k, m, 3, dtype=torch.float32).double()
        z = z * (0.9 + 0.2 * _rand(g, k, 1, 3)) + 0.08 * _randn(g, k, 1, 3) * (z * z - 1.0)
        v = z * th.sqrt() + 50.0 * _randn(g, k, 1, 3)
        live = (torch.arange(m, device="cuda")[None, :] < cnt[:, None]).double()
        U = (v * live[..., None]).sum(1) / cnt[:, None]
        c = (v - U[:, None]) * live[..., None]
        q = torch.stack([t.sum(1) for t in _monomials(c)], 1) / cnt[:, None]
        r = out[i:i + k]
        r[:, 0], r[:, 1:4], r[:, 5:31] = cnt, U, q
        r[:, 4] = (q[:, 0] + q[:, 3] + q[:, 5]) / 3.0
    if low:
        out[:, 21:] = 0.0
    return out


def _batch_workload(n, order=5):
    w = I.couette(kn=KN, ncell=100, ppc=100)
    return dict(w, nx=n, ny=1, lx=w["dx"] * n, moment_order=order)


PAIRS = [(0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2)]
SYM = [[0, 1, 2], [1, 3, 4], [2, 4, 5]]
TRI = {(0, 0, 0): 0, (0, 0, 1): 1, (0, 0, 2): 2, (0, 1, 1): 3, (0, 1, 2): 4, (0, 2, 2): 5, (1, 1, 1): 6,
       (1, 1, 2): 7, (1, 2, 2): 8, (2, 2, 2): 9}


def _normalised(mom):
    """P, T, R, W of records over the powers of theta, as lists of columns."""
    th = mom[:, 4]
    P = [mom[:, 5 + q] / th for q in range(6)]
    T = [mom[:, 11 + q] / th ** 1.5 for q in range(10)]
    R = [mom[:, 21 + q] / th ** 2 for q in range(6)]
    W = [mom[:, 27 + q] / th ** 2.5 for q in range(3)]
    return P, T, R, W


def _system(mom):
    """The moment conditions of c_i c_j and c_i |c|^2 under the cubic drift, normalised: A, b."""
    P, T, R, W = _normalised(mom)
    p = lambda i, j: P[SYM[i][j]]                                # noqa: E731
    t = lambda i, j, k: T[TRI[tuple(sorted((i, j, k)))]]         # noqa: E731
    S = [t(i, 0, 0) + t(i, 1, 1) + t(i, 2, 2) for i in range(3)]
    Q = R[0] + R[3] + R[5]
    A = torch.zeros((mom.shape[0], 9, 9), dtype=mom.dtype, device=mom.device)
    b = torch.zeros((mom.shape[0], 9), dtype=mom.dtype, device=mom.device)
    rows, rhs = [], []
    zero = torch.zeros_like(Q)
    for i, j in PAIRS:
        row = [zero] * 9
        for k in range(3):
            row[SYM[i][k]] = row[SYM[i][k]] + p(k, j)
            row[SYM[j][k]] = row[SYM[j][k]] + p(k, i)
        row[6 + i] = row[6 + i] + S[j]
        row[6 + j] = row[6 + j] + S[i]
        rows.append(torch.stack(row, 1))
        rhs.append(2.0 * EPS_HAT * R[SYM[i][j]])
    for i in range(3):
        row = [zero] * 9
        for j in range(3):
            row[SYM[i][j]] = row[SYM[i][j]] + S[j]
            for k in range(3):
                row[SYM[j][k]] = row[SYM[j][k]] + 2.0 * t(i, j, k)
            row[6 + j] = row[6 + j] + 2.0 * (R[SYM[i][j]] - 3.0 * p(i, j))
        row[6 + i] = row[6 + i] + Q - 9.0
        rows.append(torch.stack(row, 1))
        PS = p(i, 0) * S[0] + p(i, 1) * S[1] + p(i, 2) * S[2]
        rhs.append(5.0 / 3.0 * S[i] + EPS_HAT * (3.0 * W[i] - 3.0 * S[i] - 2.0 * PS))
    A, b = torch.stack(rows, 1), torch.stack(rhs, 1)
    return A, b


def _solve(A, b):
    return torch.linalg.solve(A.cpu(), b.cpu()[..., None])[..., 0].to(A.device)


def _tau(w, N, th):
    T = th * (w["mass"] / w["kB"])
    return 2.0 * w["mu_ref"] * (T / w["T_ref"]) ** w["omega"] / (N * w["fnum_over_vol"] * w["kB"] * T)


def _update_records(w, mom, y, solved):
    """Records of normalised coefficients y (zero where not solved)."""
    N, th = mom[:, 0], mom[:, 4]
    tau = _tau(w, N, th)
    rec = torch.zeros((mom.shape[0], 16), dtype=mom.dtype, device=mom.device)
    ok = solved.to(mom.dtype)
    rec[:, :6] = y[:, :6] / tau[:, None] * ok[:, None]
    rec[:, 6:9] = y[:, 6:] / (tau * th.sqrt())[:, None] * ok[:, None]
    rec[:, 9], rec[:, 10], rec[:, 11] = tau, th, torch.exp(-w["dt"] / tau)
    rec[:, 12] = EPS_HAT / (th * tau) * ok
    rec[:, 13] = (th * (1.0 - torch.exp(-2.0 * w["dt"] / tau))).sqrt()
    return rec


def _empty_records(n):
    rec = torch.zeros((n, 16), dtype=torch.float64, device="cuda")
    rec[:, 14] = float(F.CELL_EMPTY)
    return rec, torch.zeros(n, dtype=torch.int32, device="cuda")


def _prep_closure(case, seed):
    n = case["cells"]
    rec, st = _empty_records(n)
    return {"kind": "closure", "ctx": F.Context(_batch_workload(n), 1), "mom": _records(n, seed), "rec": rec, "status": st}


def _run_closure(s):
    s["ctx"].closure_solve(s["mom"], s["rec"], s["status"])
    return {"rec": s["rec"], "status": s["status"]}


# ---- networks --------------------------------------------------------------------------------
def _features(w, mom, lite):
    """Raw network inputs (padded to 32 columns for the 27-feature network)."""
    N, th = mom[:, 0], mom[:, 4]
    d6 = torch.tensor([1.0, 0, 0, 1, 0, 1], dtype=mom.dtype, device=mom.device)
    if lite:
        rho = N * w["fnum_over_vol"] * w["mass"]
        t = mom[:, 11:21]
        S = [t[:, 0] + t[:, 3] + t[:, 5], t[:, 1] + t[:, 6] + t[:, 8], t[:, 2] + t[:, 7] + t[:, 9]]
        return torch.cat([torch.stack([rho, th * (w["mass"] / w["kB"])], 1), mom[:, 1:4],
                          rho[:, None] * (mom[:, 5:11] - th[:, None] * d6),
                          torch.stack([0.5 * rho * s for s in S] + [3.0 * th, 1.0 / _tau(w, N, th)], 1)], 1)
    P, T, R, W = (torch.stack(c, 1) for c in _normalised(mom))
    tail = torch.stack([torch.full_like(N, EPS_HAT), N.log10()], 1)
    pad = torch.zeros((mom.shape[0], 5), dtype=mom.dtype, device=mom.device)
    return torch.cat([P - d6, T, R - 5.0 * d6, W, tail, pad], 1)


def _targets(w, mom, lite):
    y = _solve(*_system(mom))
    if lite:
        r = _update_records(w, mom, y, torch.ones(mom.shape[0], dtype=torch.bool, device=mom.device))
        return r[:, :9].contiguous()
    y[:, [0, 3, 5]] -= 5.0 * EPS_HAT
    return y


WIDTHS = {"nn": [32, 128, 128, 128, 16], "lite": [16, 256, 256, 256, 256, 16]}


def _unpack(net, p):
    """Weights, biases and the four scalers of a flat parameter vector."""
    w = WIDTHS[net]
    layers, o = [], 0
    for i, k in zip(w[:-1], w[1:]):
        layers.append((p[o:o + i * k].reshape(k, i), p[o + i * k:o + i * k + k]))
        o += i * k + k
    return layers, (p[o:o + w[0]], p[o + w[0]:o + 2 * w[0]], p[o + 2 * w[0]:o + 2 * w[0] + 16], p[o + 2 * w[0] + 16:])


def _forward(net, layers, x):
    h = x
    for i, (W, b) in enumerate(layers):
        h = h @ W.T + b
        if i + 1 < len(layers):
            h = torch.nn.functional.silu(h) if net == "nn" else torch.relu(h)
    return h


def _network(net, w, seed, fitted):
    """Flat FP32 parameters: scalers from a sample of records, Glorot weights and zero biases
    as training starts; fitted: the output layer by least squares, so that the network
    predicts as a trained one does."""
    lite = net == "lite"
    mom = _records(16384, 7001)
    x, y = _features(w, mom, lite), _targets(w, mom, lite)
    xm, xs = x.mean(0), x.std(0, unbiased=False)
    xs = torch.where(xs > 1e-6 * xm.abs().clamp(min=1.0), xs, torch.ones_like(xs))
    one, zero = torch.ones(7, dtype=x.dtype, device="cuda"), torch.zeros(7, dtype=x.dtype, device="cuda")
    ym, ys = torch.cat([y.mean(0), zero]), torch.cat([y.std(0, unbiased=False), one])
    g = _gen(seed + 1)
    layers, wd = [], WIDTHS[net]
    for i, k in zip(wd[:-1], wd[1:]):
        W = (2.0 * _rand(g, k, i) - 1.0) * math.sqrt(6.0 / (i + k))
        if k == 16:
            W[9:] = 0.0
        if i == 32:
            W[:, 27:] = 0.0
        layers.append([W.float().double(), torch.zeros(k, dtype=torch.float64, device="cuda")])
    if fitted:
        h = _forward(net, layers[:-1] + [[torch.eye(wd[-2], dtype=x.dtype, device="cuda"), 0.0]], (x - xm) / xs)
        h = torch.nn.functional.silu(h) if net == "nn" else torch.relu(h)
        h = torch.cat([h, torch.ones((h.shape[0], 1), dtype=h.dtype, device="cuda")], 1).cpu().numpy()
        t = ((y - ym[:9]) / ys[:9]).cpu().numpy()
        c = np.linalg.solve(h.T @ h + 1e-3 * np.eye(h.shape[1]), h.T @ t)
        layers[-1][0][:9] = torch.from_numpy(c[:-1].T.copy()).cuda()
        layers[-1][1][:9] = torch.from_numpy(c[-1].copy()).cuda()
    parts = [t.reshape(-1) for l in layers for t in l] + [xm, xs, ym, ys]
    return torch.cat(parts).float()


def _learned(case, seed):
    net, n = case["kind"], case["cells"]
    w = _batch_workload(n, 3 if net == "lite" else 5)
    return w, _network(net, w, seed, True), _records(n, seed, low=net == "lite")


def _prep_learned(case, seed):
    w, params, mom = _learned(case, seed)
    ctx = F.Context(w, 1)
    net = F.Network(ctx) if case["kind"] == "nn" else F.LiteNetwork(ctx)
    net.load(params)
    rec, st = _empty_records(case["cells"])
    tol = (0.05, 0.05) if case.get("checked") else (math.inf, 0.0)
    return {"kind": case["kind"], "ctx": ctx, "net": net, "mom": mom, "rec": rec, "status": st,
            "tol": tol + (case["relax"],)}


def _run_learned(s):
    s["net"].closure(s["mom"], s["rec"], s["status"], *s["tol"])
    return {"rec": s["rec"], "status": s["status"]}


def _train_data(case, seed):
    lite = case["net"] == "lite"
    w = _batch_workload(1)
    mom = _records(case["batch"], seed)
    mom[:, 0].clamp_(min=5.0)
    feats = _features(w, mom, lite).float()
    tg = sys = None
    if case["loss"] == "mse":
        tg = torch.zeros((case["batch"], 16), dtype=torch.float32, device="cuda")
        tg[:, :9] = _targets(w, mom, lite).float()
    else:
        A, b = _system(mom)
        sys = torch.cat([A.reshape(-1, 81), b], 1)
    return w, _network(case["net"], w, seed, False), feats, tg, sys


def _prep_train(case, seed):
    w, params, feats, tg, sys = _train_data(case, seed)
    ctx = F.Context(w, 1)
    net = (F.LiteNetwork if case["net"] == "lite" else F.Network)(ctx, case["batch"])
    return {"kind": "train", "net": net, "lite": case["net"] == "lite", "params": params, "m": torch.zeros_like(params),
            "v": torch.zeros_like(params), "t": 0, "feats": feats.contiguous(), "tg": tg, "sys": sys,
            "loss_kind": F.LOSS_MSE if case["loss"] == "mse" else F.LOSS_RESIDUAL,
            "loss": torch.zeros(1, dtype=torch.float32, device="cuda")}


def _run_train(s):
    s["t"] += 1
    B = s["feats"].shape[0]
    if s["lite"]:
        s["net"].train_step(s["params"], s["m"], s["v"], s["t"], LR, s["feats"], s["tg"], B, s["loss"])
    else:
        s["net"].train_step(s["params"], s["m"], s["v"], s["t"], LR, s["feats"], s["tg"], s["sys"], B,
                            s["loss_kind"], s["loss"])
    return {"params": s["params"], "m": s["m"], "v": s["v"], "loss": s["loss"]}


# ---- differentiation -------------------------------------------------------------------------
def _grad_data(case, seed):
    """Velocities of cells of lo .. hi particles, each cell a skewed anisotropic Gaussian (the
    particle counts are the case's, the same for every seed: they are the outputs' lengths)."""
    g = _gen(seed)
    nc = case["cells"]
    dt = torch.float32 if case["precision"] == "f32" else torch.float64
    cnt = torch.randint(case["lo"], case["hi"] + 1, (nc,), generator=_gen(7002), device="cuda")
    off = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), cnt.cumsum(0)])
    cell = torch.arange(nc, device="cuda").repeat_interleave(cnt)
    n = int(off[-1])
    s = math.sqrt(I.KB / I.MASS_AR * 273.0)
    z = _randn(g, n, 3)
    a, k, u = 0.8 + 0.4 * _rand(g, nc, 3), 0.1 * _randn(g, nc, 3), 0.5 * _randn(g, nc, 3)
    v = ((z * a[cell] + k[cell] * (z * z - 1.0) + u[cell]) * s).to(dt)
    w = dict(_batch_workload(nc), precision=case["precision"])
    gy = _randn(g, nc, 9)
    return w, v, off, cell, cnt, gy


def _prep_grad(case, seed):
    w, v, off, _, _, gy = _grad_data(case, seed)
    ctx = F.Context(w, int(v.shape[0]))
    return {"kind": "grad", "ctx": ctx, "v": [v[:, i].contiguous().requires_grad_() for i in range(3)],
            "off": off.to(torch.int32), "gy": gy}


def _run_grad(s):
    y = ExactClosure.apply(*s["v"], s["ctx"], s["off"])
    gx = torch.autograd.grad(y, s["v"], s["gy"])
    return {"y": y.detach(), "gx": gx[0], "gy": gx[1], "gz": gx[2]}


# ---- 64-bit references -----------------------------------------------------------------------
def _exact_closure(case, seed):
    w, mom = _batch_workload(case["cells"]), _records(case["cells"], seed)
    enough = mom[:, 0] >= w["n_min"]
    A, b = _system(mom)
    eye = torch.eye(9, dtype=A.dtype, device=A.device)
    y = _solve(torch.where(enough[:, None, None], A, eye), b)
    rec = _update_records(w, mom, y, enough)
    return {"rec": rec, "status": None}


def _exact_learned(case, seed):
    net = case["kind"]
    w, params, mom = _learned(case, seed)
    p = params.double()
    layers, (xm, xs, ym, ys) = _unpack(net, p)
    enough = mom[:, 0] >= w["n_min"]
    out = []
    for m in mom.split(100000):
        out.append(_forward(net, layers, (_features(w, m, net == "lite") - xm) / xs) * ys + ym)
    y = torch.cat(out)[:, :9]
    th = mom[:, 4]
    if net == "lite":
        tau = _tau(w, mom[:, 0], th)
        y = torch.cat([y[:, :6] * tau[:, None], y[:, 6:] * (tau * th.sqrt())[:, None]], 1)
    else:
        y[:, [0, 3, 5]] += 5.0 * EPS_HAT
    if case.get("checked"):
        A, b = _system(mom)
        r = (A @ y[..., None])[..., 0] - b
        bad = torch.nonzero(~(r.norm(dim=1) <= 0.05 + 0.05 * b.norm(dim=1)) & enough)[:, 0]
        y[bad] = _solve(A[bad], b[bad])
    return {"rec": _status_free(_update_records(w, mom, y, enough)), "status": None}


def _status_free(rec):
    rec[:, 14] = float(F.CELL_NN)
    return rec


def _exact_train(case, seed):
    w, params, feats, tg, sys = _train_data(case, seed)
    net = case["net"]
    p = params.double().cpu().requires_grad_()
    layers, (xm, xs, ym, ys) = _unpack(net, p)
    B = case["batch"]
    y = _forward(net, layers, (feats.double().cpu() - xm.detach()) / xs.detach())[:, :9]
    if case["loss"] == "mse":
        t = (tg.double().cpu()[:, :9] - ym.detach()[:9]) / ys.detach()[:9]
        loss = ((y - t) ** 2).sum() / B
    else:
        s = sys.cpu()
        y = y * ys.detach()[:9] + ym.detach()[:9]
        y = y + 5.0 * EPS_HAT * torch.tensor([1.0, 0, 0, 1, 0, 1, 0, 0, 0], dtype=y.dtype)
        r = torch.bmm(s[:, :81].reshape(-1, 9, 9), y[..., None])[..., 0] - s[:, 81:]
        loss = (r * r).sum() / B
    loss.backward()
    g = p.grad
    m, v = 0.1 * g, 0.001 * g * g
    with torch.no_grad():
        q = p - LR * g / (g.abs() + 1e-8)
    return {"params": q, "m": m, "v": v, "loss": loss.detach().reshape(1)}


def _exact_grad(case, seed):
    w, v, _, cell, cnt, gy = _grad_data(case, seed)
    nc = case["cells"]
    v = v.double().requires_grad_()
    N = cnt.double()

    def mean(x):
        return torch.zeros((nc,) + x.shape[1:], dtype=x.dtype, device=x.device).index_add(0, cell, x) / N[:, None]

    c = v - mean(v)[cell]
    q = mean(torch.stack(_monomials(c), 1))
    th = (q[:, 0] + q[:, 3] + q[:, 5]) / 3.0
    mom = torch.cat([N[:, None], torch.zeros((nc, 3), dtype=q.dtype, device=q.device), th[:, None], q], 1)
    enough = N >= w["n_min"]
    A, b = _system(mom)
    y = _solve(A, b)
    y = _update_records(w, mom, y, enough)[:, :9]
    (gv,) = torch.autograd.grad(y, v, gy)
    return {"y": y.detach(), "gx": gv[:, 0], "gy": gv[:, 1], "gz": gv[:, 2]}


def _np_moments(v, off):
    """Records [ncell][32] of velocities v [3][n] grouped by off (numpy, FP64)."""
    nc, n = off.shape[0] - 1, np.diff(off).astype(np.float64)
    cell = np.repeat(np.arange(nc), np.diff(off))
    inv = 1.0 / np.maximum(n, 1.0)
    mom = np.zeros((nc, 32))
    mom[:, 0] = n
    U = np.stack([np.bincount(cell, x, nc) * inv for x in v])
    mom[:, 1:4] = U.T
    c = np.stack([x - u[cell] for x, u in zip(v, U)], -1)
    for i, q in enumerate(_monomials(c)):
        mom[:, 5 + i] = np.bincount(cell, q, nc) * inv
    mom[:, 4] = (mom[:, 5] + mom[:, 8] + mom[:, 10]) / 3.0
    return mom


def _np_sums(mom):
    """One sample's raw sums [ncell][16] of moment records."""
    N, U, P, T = mom[:, 0], mom[:, 1:4], mom[:, 5:11], mom[:, 11:21]
    out = np.zeros((mom.shape[0], 16))
    out[:, 0] = N
    out[:, 1:4] = N[:, None] * U
    for q, (i, j) in enumerate(PAIRS):
        out[:, 4 + q] = N * (P[:, q] + U[:, i] * U[:, j])
    U2 = (U * U).sum(1)
    tr = P[:, 0] + P[:, 3] + P[:, 5]
    for i in range(3):
        S = sum(T[:, TRI[tuple(sorted((i, k, k)))]] for k in range(3))
        PU = sum(P[:, SYM[i][k]] * U[:, k] for k in range(3))
        out[:, 10 + i] = N * (S + 2.0 * PU + U[:, i] * (tr + U2))
    out[:, 13] = 1.0
    return out


def _exact_resort(case, seed):
    _, st, _ = _resort_state(case, seed)
    order = np.argsort(st["key"], kind="stable")
    nc = case["cells"] ** 2
    off = np.concatenate([[0], np.cumsum(np.bincount(st["key"], minlength=nc))])
    v = np.stack([st[k][order].astype(np.float64) for k in ("vx", "vy", "vz")])
    mom = _np_moments(v, off)
    out = {k: st[k][order].astype(np.float64) for k in ("x", "y", "vx", "vy", "vz")}
    out.update(pid=None, key=None, offsets=None, perm=None, mom=mom, samp=_np_sums(mom))
    return out


def _np_philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 (Salmon et al., SC'11) on arrays of counters, key = seed low / high."""
    u, low, s32 = np.uint64, np.uint64(0xFFFFFFFF), np.uint64(32)
    x = [np.broadcast_to(np.asarray(v, dtype=u), c0.shape) for v in (c0, c1, c2, c3)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        p, q = u(0xD2511F53) * x[0], u(0xCD9E8D57) * x[2]
        x = [(q >> s32) ^ x[1] ^ u(k0), q & low, (p >> s32) ^ x[3] ^ u(k1), p & low]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return [(a.astype(np.float64) + 0.5) * 2.0 ** -32 for a in x]


def _np_fly(w, p, v, pid, step, store):
    """Free flight over dt with diffuse walls; p [d][n], v [3][n] in place."""
    d = p.shape[0]
    lo, hi = [w["x0"], w["y0"]], [w["x0"] + w["lx"], w["y0"] + w["ly"]]
    todo = np.arange(p.shape[1])
    rem = np.full(todo.shape[0], float(w["dt"]))
    for bounce in range(w["max_bounces"] + 1):
        q, u = p[:, todo], v[:, todo]
        e = q + u[:d] * rem
        wall, th = np.full(todo.shape[0], -1), np.zeros(todo.shape[0])
        for k in range(2 * d):
            a, face = k // 2, (lo, hi)[k % 2][k // 2]
            out = (e[a] < face) & (u[a] < 0.0) if k % 2 == 0 else (e[a] > face) & (u[a] > 0.0)
            t = np.maximum((face - q[a]) / np.where(u[a] == 0.0, 1.0, u[a]), 0.0)
            first = out & ((wall < 0) | (t < th))
            wall, th = np.where(first, k, wall), np.where(first, t, th)
        hit = wall >= 0
        p[:, todo[~hit]] = e[:, ~hit]
        if bounce == w["max_bounces"]:
            for a in range(d):
                p[a, todo[hit]] = np.clip(e[a, hit], lo[a], hi[a])
            break
        todo, wall, th, rem = todo[hit], wall[hit], np.minimum(th[hit], rem[hit]), rem[hit]
        if todo.size == 0:
            break
        q, u = p[:, todo] + v[:d, todo] * th, v[:, todo]
        r = _np_philox(pid[todo].astype(np.uint64), step, 4, bounce, w["seed"])
        rt, uw = w["R"] * np.asarray(w["T_wall"])[wall], np.asarray(w["u_wall"])[wall].T
        vn = np.sqrt(-2.0 * rt * np.log(r[0]))
        rr = np.sqrt(-2.0 * np.log(r[1]) * rt)
        ta, tb = rr * np.cos(2 * np.pi * r[2]), rr * np.sin(2 * np.pi * r[2])
        sgn = np.where(wall % 2 == 0, 1.0, -1.0)
        onx = wall < 2
        u = np.stack([np.where(onx, sgn * vn, uw[0] + ta), np.where(onx, uw[1] + ta, sgn * vn), uw[2] + tb])
        for a in range(d):
            q[a] = np.where(wall == 2 * a, lo[a], np.where(wall == 2 * a + 1, hi[a], q[a]))
        p[:, todo], v[:, todo] = q, store(u)
        rem = rem - th
    p[:] = store(p)


def _exact_loop(case, seed):
    """Three steps (one eager, two replayed) of the box loop, stored in the case's precision."""
    w = _box(case, seed)
    two_d = w["geometry"] != "couette1d"
    if w["nx"] * w["ny"] * w["ppc"] > 1200000:
        return None
    st = _box_state(w, seed)
    dt = np.float32 if w["precision"] == "f32" else np.float64
    store = lambda a: a.astype(dt).astype(np.float64)            # noqa: E731
    p = np.stack([st[k].astype(np.float64) for k in (("x", "y") if two_d else ("x",))])
    v = np.stack([st[k].astype(np.float64) for k in ("vx", "vy", "vz")])
    pid, nc = st["pid"], w["nx"] * w["ny"]
    samp = np.zeros((nc, 16))

    def keys():
        k = [np.clip(np.floor((p[a] - o) * (1.0 / h)), 0, m - 1).astype(np.int64)
             for a, (o, h, m) in enumerate([(w["x0"], w["dx"], w["nx"]), (w["y0"], w["dy"], w["ny"])][:len(p)])]
        return k[0] + (k[1] * w["nx"] if two_d else 0)

    key = keys()
    for s in range(3):
        order = np.argsort(key, kind="stable")
        p, v, pid, key = p[:, order], v[:, order], pid[order], key[order]
        off = np.concatenate([[0], np.cumsum(np.bincount(key, minlength=nc))])
        mom = _np_moments(v, off)
        if case["sample"]:
            samp += _np_sums(mom)
        m = torch.from_numpy(mom)
        enough = m[:, 0] >= w["n_min"]
        A, b = _system(m)
        A = torch.where(enough[:, None, None], A, torch.eye(9, dtype=A.dtype))
        y = _solve(A, torch.where(enough[:, None], b, torch.zeros_like(b)))
        live = (mom[:, 0] > 1) & (mom[:, 4] > 0)
        rec = _update_records(w, m, y, enough).numpy()
        rec[~live] = 0.0
        rec[~live, 11] = 1.0
        rec[~live, 10] = mom[~live, 4]
        r = rec[key].T
        c = v - mom[key, 1:4].T
        th, E, tau = r[10], r[11], r[9]
        c2 = (c * c).sum(0)
        S = np.stack([sum(mom[:, 11 + TRI[tuple(sorted((i, k, k)))]] for k in range(3))[key] for i in range(3)])
        N = np.stack([sum(r[SYM[i][k]] * c[k] for k in range(3)) + r[6 + i] * (c2 - 3.0 * th)
                      - r[12] * (c[i] * c2 - S[i]) for i in range(3)])
        u = _np_philox(pid.astype(np.uint64), s, 3, 0, w["seed"])
        r0, r1 = np.sqrt(-2.0 * np.log(u[0])), np.sqrt(-2.0 * np.log(u[2]))
        z = np.stack([r0 * np.cos(2 * np.pi * u[1]), r0 * np.sin(2 * np.pi * u[1]), r1 * np.cos(2 * np.pi * u[3])])
        cs = c * E + (1.0 - E) * tau * N + r[13] * z
        inv = 1.0 / np.maximum(mom[:, 0], 1.0)
        cb = np.stack([np.bincount(key, x, nc) * inv for x in cs])
        with np.errstate(all="ignore"):
            if w["conserve"] == "exact":
                e2 = np.bincount(key, (cs * cs).sum(0), nc) * inv - (cb * cb).sum(0)
                sc = np.sqrt(3.0 * mom[:, 4] / e2)
            else:
                nn, cn = np.bincount(key, (N * N).sum(0), nc) * inv, np.bincount(key, (c * N).sum(0), nc) * inv
                t, e, q = rec[:, 9], rec[:, 11], rec[:, 10]
                sc = 1.0 / np.sqrt(1.0 + t / (3.0 * q) * (t * (1 - e) ** 2 * nn + 2.0 * (e - e * e) * cn))
            sc = np.where(np.isfinite(sc) & (sc > 0), sc, 1.0)
        v = np.where(live[key], store((cs - cb[:, key]) * sc[key] + mom[key, 1:4].T), v)
        _np_fly(w, p, v, pid, s, store)
        key = keys()
    out = {"x": p[0], "vx": v[0], "vy": v[1], "vz": v[2], "pid": None, "key": None, "offsets": None, "mom": mom,
           "rec": rec, "status": None, "samp": samp}
    if two_d:
        out["y"] = p[1]
    return out


_PREPARE = {"loop": _prep_loop, "cylinder": _prep_cylinder, "resort": _prep_resort, "closure": _prep_closure,
            "nn": _prep_learned, "lite": _prep_learned, "train": _prep_train, "grad": _prep_grad}
_RUN = {"loop": _run_loop, "cylinder": _run_cylinder, "resort": _run_resort, "closure": _run_closure,
        "nn": _run_learned, "lite": _run_learned, "train": _run_train, "grad": _run_grad}
_EXACT = {"loop": _exact_loop, "resort": _exact_resort, "closure": _exact_closure, "nn": _exact_learned,
          "lite": _exact_learned, "train": _exact_train, "grad": _exact_grad}
