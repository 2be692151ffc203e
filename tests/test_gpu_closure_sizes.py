"""The exact and the checked closure at the edges of a wave (64 cells).  A cell's result may
not depend on the lanes beside it (which decide what row swaps a wave skips), on its place in
the wave, on whether its records are 16-byte aligned or on what lies behind the last cell: the
bits must be the same for rolled records, for records eight bytes off alignment, and for each
cell in a context of its own.  Statuses are the oracle's."""
import numpy as np
import pytest
import torch

from oracle import mlp_oracle as M
from oracle import oracle as O
from paper_2606_15622_amd import inputs as I

pytestmark = pytest.mark.gpu


def fp():
    from paper_2606_15622_amd import fpgpu
    fpgpu.load()
    return fpgpu


def records(n, seed):
    rng = np.random.default_rng(seed)
    counts = rng.choice([0, 1, 5, 6, 8, 12, 40, 300], n)   # few particles: pivots off the diagonal
    vx, vy, vz, off = I.mixture_cells(counts, seed=seed)
    mom = O.moments(off, vx, vy, vz)
    if n > 8:
        mom[3, 12] = np.nan
        mom[5, 4] = 0.0
    return mom


def solve(F, w, mom, shift, pd=None, relax=1.0):
    n = mom.shape[0]
    ctx = F.Context(dict(w, nx=n, ny=1, lx=w["dx"] * n), 1)
    buf = torch.empty(n * 32 + shift, dtype=torch.float64, device="cuda")
    md = buf[shift:].view(n, 32)
    md.copy_(torch.from_numpy(np.ascontiguousarray(mom)))
    guard = 7
    rec = torch.full((n + guard, 16), 2.5, dtype=torch.float64, device="cuda")
    st = torch.full((n + guard,), -9, dtype=torch.int32, device="cuda")
    if pd is None:
        ctx.closure_solve(md, rec, st)
    else:
        net = F.Network(ctx, 0)
        net.load(pd)
        net.closure(md, rec, st, 0.0, 0.3, relax)
    torch.cuda.synchronize()
    assert bool((rec[n:] == 2.5).all()) and bool((st[n:] == -9).all())
    return rec[:n].cpu().numpy(), st[:n].cpu().numpy()


@pytest.mark.parametrize("n", [1, 63, 64, 65, 131])
@pytest.mark.parametrize("learned", [False, True])
def test_a_cell_does_not_depend_on_its_wave(n, learned):
    F = fp()
    w = I.couette(ncell=100, precision="f64", eps_hat=0.01)
    mom = records(n, n)
    pd = None
    if learned:
        rng = np.random.default_rng(5)
        d = {name: 0.05 * rng.standard_normal(shp) for name, shp in M.SHAPES}
        d["x_std"], d["y_std"] = np.ones_like(d["x_std"]), np.ones_like(d["y_std"])
        pd = torch.from_numpy(M.pack(d).astype(np.float32)).cuda()
    relax = 0.4 if learned else 1.0
    rec, st = solve(F, w, mom, 0, pd, relax)
    if not learned:
        np.testing.assert_array_equal(st, O.closure(dict(w, nx=n, ny=1), mom)[1])
    off_rec, off_st = solve(F, w, mom, 1, pd, relax)
    np.testing.assert_array_equal(rec, off_rec)
    np.testing.assert_array_equal(st, off_st)
    r_rec, r_st = solve(F, w, np.roll(mom, 17, axis=0), 0, pd, relax)
    np.testing.assert_array_equal(np.roll(rec, 17, axis=0), r_rec)
    np.testing.assert_array_equal(np.roll(st, 17), r_st)
    for i in range(0, n, 9):
        one, s1 = solve(F, w, mom[i:i + 1], 0, pd, relax)
        np.testing.assert_array_equal(rec[i:i + 1], one)
        assert s1[0] == st[i]
