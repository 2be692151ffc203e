"""Moments at the cell populations around the rounds in which moments_kernel takes the particles
beyond the eight a lane holds in registers: eight at a time for the sums (the next round from
16 lanes' worth on), six for the moments (from 14, 20 on); for every group width, against the
oracle with the bounds of the general tests."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2606_15622_amd import inputs as I
from test_gpu_rebin import fp, moment_scale

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("lanes", [4, 8, 16, 32, 64])
def test_moments_around_the_later_rounds(prec, lanes):
    F = fp()
    edges = [k * lanes + d for k in (8, 14, 16, 20, 24) for d in (-1, 0, 1)]
    counts = np.random.default_rng(lanes).permutation(np.concatenate([edges, edges, [0, 1, 3 * lanes]]))
    nc = counts.size
    vx, vy, vz, off = I.mixture_cells(counts, seed=lanes)
    v = [a.astype(np.float32 if prec == "f32" else np.float64) for a in (vx, vy, vz)]
    w = dict(I.couette(ncell=nc, precision=prec), lanes=lanes)
    ctx = F.Context(w, v[0].size)
    z = np.zeros_like(v[0])
    p = F.Particles.from_numpy(w, dict(x=z, y=z, vx=v[0], vy=v[1], vz=v[2], pid=np.arange(z.size, dtype=np.uint32),
                                       key=np.repeat(np.arange(nc), counts).astype(np.int32)))
    mom = torch.full((nc, 32), -7.0, dtype=torch.float64, device="cuda")
    ctx.moments(p, torch.tensor(off, dtype=torch.int32, device="cuda"), mom)
    torch.cuda.synchronize()
    o, g = O.moments(off, *(a.astype(np.float64) for a in v)), mom.cpu().numpy()
    np.testing.assert_array_equal(g[:, 0], o[:, 0])
    assert np.all(np.abs(g - o) <= 1e-10 * moment_scale(o))
