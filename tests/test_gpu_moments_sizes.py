"""Moments and their reverse mode at the cell populations where the kernels change: the
particles a lane holds in registers (eight), a remainder beyond them in rounds of four, and
cells of very different sizes side by side, for every group width; against the oracle (the
bounds of the general tests)."""
import numpy as np
import pytest
import torch

from oracle import diff_oracle as D
from oracle import oracle as O
from paper_2606_15622_amd import inputs as I
from test_gpu_rebin import fp, moment_scale

pytestmark = pytest.mark.gpu


def counts_around(lanes, seed):
    rng = np.random.default_rng(seed)
    edges = [8 * lanes + d for d in (-1, 0, 1)] + [12 * lanes + d for d in (-1, 0, 1)] + [29 * lanes + 3]
    return np.concatenate([rng.choice([5, lanes, 2 * lanes + 1] + edges, 150), [0, 1, 0, 6]])


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("lanes", [4, 8, 16, 32, 64])
def test_moments_around_the_register_cache(prec, lanes):
    F = fp()
    counts = counts_around(lanes, lanes)
    nc = counts.size
    vx, vy, vz, off = I.mixture_cells(counts, seed=lanes)
    dt = np.float32 if prec == "f32" else np.float64
    v = [a.astype(dt) for a in (vx, vy, vz)]
    w = dict(I.couette(ncell=nc, precision=prec), lanes=lanes)
    ctx = F.Context(w, v[0].size)
    z = np.zeros_like(v[0])
    p = F.Particles.from_numpy(w, dict(x=z, y=z, vx=v[0], vy=v[1], vz=v[2],
                                       pid=np.arange(z.size, dtype=np.uint32),
                                       key=np.repeat(np.arange(nc), counts).astype(np.int32)))
    offd = torch.tensor(off, dtype=torch.int32, device="cuda")
    mom = torch.full((nc, 32), -7.0, dtype=torch.float64, device="cuda")
    ctx.moments(p, offd, mom)
    torch.cuda.synchronize()
    o = O.moments(off, *(a.astype(np.float64) for a in v))
    g = mom.cpu().numpy()
    np.testing.assert_array_equal(g[:, 0], o[:, 0])
    assert np.all(np.abs(g - o) <= 1e-10 * moment_scale(o))


@pytest.mark.parametrize("lanes", [4, 8, 16, 32, 64])
def test_reverse_mode_around_the_register_cache(lanes):
    F = fp()
    from paper_2606_15622_amd.autograd import ExactClosure
    counts = np.maximum(counts_around(lanes, lanes + 1), 12)
    vx, vy, vz, off = I.mixture_cells(counts, seed=lanes + 1)
    v = np.stack([vx, vy, vz], 1)
    nc = counts.size
    w = I.couette(ncell=nc, precision="f64", eps_hat=0.01)
    ctx = F.Context(dict(w, lanes=lanes), v.shape[0])
    vd = [torch.tensor(v[:, a], device="cuda", requires_grad=True) for a in range(3)]
    offd = torch.tensor(off, dtype=torch.int32, device="cuda")
    th = I.KB / I.MASS_AR * 273.0
    wts = np.random.default_rng(12).standard_normal((nc, 9)) * np.array([1.0] * 6 + [np.sqrt(th)] * 3)
    y = ExactClosure.apply(vd[0], vd[1], vd[2], ctx, offd)
    (y * torch.tensor(wts, device="cuda")).sum().backward()
    g = np.stack([t.grad.cpu().numpy() for t in vd], 1)
    vt = torch.tensor(v, requires_grad=True)
    yo = D.coefficients(vt, off, w)
    (yo * torch.tensor(wts)).sum().backward()
    go = vt.grad.numpy()
    assert np.abs(g - go).max() <= 1e-8 * np.abs(go).max()
    assert np.linalg.norm(g - go) <= 1e-9 * np.linalg.norm(go)
