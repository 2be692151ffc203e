"""The LITE closure at the cell counts where its launch changes: less than a wave, the last
count of four-wave workgroups (32,768 cells) and the first of eight-wave ones, and workgroups
that take a second pass.  Cells are independent, so every row must be the same bits as in a
small context; and on third-order records the one-kernel closure must give the bits of the
network kernel followed by the check kernel (a fifth-order context, unchecked)."""
import math

import numpy as np
import pytest
import torch

from oracle import lite_oracle as L
from paper_2606_15622_amd import inputs as I

pytestmark = pytest.mark.gpu


def fp():
    from paper_2606_15622_amd import fpgpu
    fpgpu.load()
    return fpgpu


def records(n, seed):
    """Third-order records with empty, single-particle, few-particle and non-finite cells."""
    rng = np.random.default_rng(seed)
    m = np.zeros((n, 32))
    th = 5e4 * rng.uniform(0.5, 2.0, n)
    m[:, 0] = rng.integers(0, 200, n)
    m[:, 1:4] = 100.0 * rng.standard_normal((n, 3))
    m[:, 4] = th
    m[:, 5:11] = th[:, None] * (np.array([1, 0, 0, 1, 0, 1]) + 0.1 * rng.standard_normal((n, 6)))
    m[:, 11:21] = th[:, None] ** 1.5 * 0.1 * rng.standard_normal((n, 10))
    if n > 8:
        m[1, 0], m[2, 4], m[3, 4], m[4, 7], m[5, 12] = 1.0, 0.0, -1.0, np.nan, np.inf
    return torch.from_numpy(m).cuda()


def params(seed):
    rng = np.random.default_rng(seed)
    parts = []
    for name, shp in L.SHAPES:
        if name[0] == "W":
            p = rng.standard_normal(shp) * np.sqrt(2.0 / shp[1])
        elif name[0] == "b":
            p = rng.standard_normal(shp) * 0.05
        elif name == "x_mean":
            p = np.zeros(shp)
        elif name == "x_std":
            p = np.array([1e-6, 300, 100, 100, 100] + [1e-2] * 6 + [1.0] * 3 + [1.5e5, 1e9])
        else:
            p = np.full(shp, 1e5)
        if shp[0] == 16 and name[0] in "Wb" and name[1] == "5":
            p[9:] = 0.0
        parts.append(np.asarray(p).ravel())
    return torch.from_numpy(np.concatenate(parts).astype(np.float32)).cuda()


def context(F, n, order):
    w = I.couette(ncell=100)
    return F.Context(dict(w, nx=n, ny=1, lx=w["dx"] * n, moment_order=order), 1)


def run(F, mom, order, pd, relax, prev, outputs=False):
    n = mom.shape[0]
    net = F.LiteNetwork(context(F, n, order))
    net.load(pd)
    if outputs:
        y = torch.full((n, 16), 7.0, device="cuda")
        net.infer(mom, y)
        return y
    rec, st = prev.clone(), torch.full((n,), -1, dtype=torch.int32, device="cuda")
    net.closure(mom, rec, st, math.inf, 0.0, relax)
    return rec, st


@pytest.mark.parametrize("n", [1, 31, 129, 32768, 32769, 65536 + 33])
def test_rows_do_not_depend_on_the_launch(n):
    F = fp()
    mom, pd = records(n, n), params(3)
    prev = torch.zeros((n, 16), dtype=torch.float64, device="cuda")
    prev[:, :9] = 1e5
    prev[::2, 14] = float(F.CELL_EMPTY)
    for relax in (1.0, 0.2):
        rec, st = run(F, mom, 3, pd, relax, prev)
        rec5, st5 = run(F, mom, 5, pd, relax, prev)
        torch.cuda.synchronize()
        assert torch.equal(st, st5) and torch.equal(rec.nan_to_num(), rec5.nan_to_num())
        assert n < 100 or {F.CELL_NN, F.CELL_EMPTY, F.CELL_FEW, F.CELL_NONFINITE} <= set(st.tolist())
    y = run(F, mom, 3, pd, 1.0, prev, outputs=True)
    for i in range(0, n, 9973):
        k = min(n, i + 61)
        part = run(F, mom[i:k].contiguous(), 3, pd, 1.0, prev, outputs=True)
        torch.cuda.synchronize()
        assert torch.equal(y[i:k].nan_to_num(), part.nan_to_num())
        r, s = run(F, mom[i:k].contiguous(), 3, pd, 0.2, prev[i:k].contiguous())
        assert torch.equal(rec[i:k].nan_to_num(), r.nan_to_num()) and torch.equal(st[i:k], s)


def test_a_network_that_is_not_finite_takes_the_langevin_drift():
    F = fp()
    n = 300
    mom, pd = records(n, 5), params(4)
    pd[F.LITE_TRAIN - 16] = float("nan")   # the first output's bias
    prev = torch.zeros((n, 16), dtype=torch.float64, device="cuda")
    rec, st = run(F, mom, 3, pd, 1.0, prev)
    torch.cuda.synchronize()
    solv = (mom[:, 0] >= 5) & torch.isfinite(mom).all(1) & (mom[:, 4] > 0)
    assert bool((st[solv] == F.CELL_SINGULAR).all()) and bool((rec[solv][:, :9] == 0).all())
    assert bool((rec[solv][:, 9] > 0).all())
