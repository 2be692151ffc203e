"""The re-sort at the cell populations where its gather changes (one, two or all positions a
lane; the shift to an aligned slot; a second round), and both sorts at the cell counts where
their scans change (the one-kernel scan, the tiles of 1024 cells, the wide tiles), against
the stable counting sort: offsets, permutation and records bit for bit, moments as in the
general test of the re-sort."""
import numpy as np
import pytest
import torch

from paper_2606_15622_amd import inputs as I
from test_gpu_rebin import fp, run_rebin

pytestmark = pytest.mark.gpu


def state(w, counts, rng, far=0):
    """Particles with the given number in each cell (of a grid in row-major order), each
    coming from its cell or a neighbour, grouped by where they come from."""
    nx, ny = w["nx"], w["ny"]
    nc, n = nx * ny, int(counts.sum())
    key = rng.permutation(np.repeat(np.arange(nc), counts)).astype(np.int32)
    old = (np.clip(key % nx + rng.integers(-1, 2, n), 0, nx - 1)
           + nx * np.clip(key // nx + rng.integers(-1, 2, n), 0, ny - 1))
    if far:
        old[rng.choice(n, far, replace=False)] = rng.integers(0, nc, far)
    order = np.argsort(old, kind="stable")
    off0 = np.concatenate([[0], np.cumsum(np.bincount(old, minlength=nc))]).astype(np.int32)
    dt = np.float32 if w["precision"] == "f32" else np.float64
    s = {k: rng.standard_normal(n).astype(dt) * 300 for k in ("vx", "vy", "vz")}
    s.update({k: rng.random(n).astype(dt) for k in ("x", "y")})
    s.update(pid=np.arange(n, dtype=np.uint32), key=key[order])
    return s, off0


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("lanes", [8, 32, 64])
@pytest.mark.parametrize("far", [0, 40])
def test_populations_around_the_gathers_rounds(prec, lanes, far):
    F = fp()
    rng = np.random.default_rng(lanes + far)
    w = dict(I.cavity(ncell=24, ppc=100, precision=prec), lanes=lanes)
    g = min(lanes, 32) if lanes != 64 else 64
    edges = [0, 1] + [k * g + d for k in (1, 2, 3, 4, 5, 6) for d in (-1, 0, 1)]
    # whole stretches of small cells, of larger ones, and both side by side in a wave
    counts = np.concatenate([rng.choice([0, 1, g - 1, g], 150), rng.choice([0, g + 1, 2 * g - 1, 2 * g], 150),
                             rng.choice(edges, 24 * 24 - 300)])
    s, off0 = state(w, counts, rng, far)
    run_rebin(F, w, s, off0)


@pytest.mark.parametrize("nx,ny", [(565, 29), (1024, 17), (1023, 17), (19457, 1), (1449, 1449)])
def test_cell_counts_around_the_scans_tiles(nx, ny):
    F = fp()
    rng = np.random.default_rng(nx)
    w = I.cavity(ncell=8, ppc=4, precision="f32")
    w = dict(w, nx=nx, ny=ny, lx=nx * w["dx"], ly=ny * w["dy"])
    nc, n = nx * ny, 60_000
    counts = np.bincount(rng.integers(0, nc, n), minlength=nc)
    s, off0 = state(w, counts, rng, 500)
    ctx = F.Context(w, n)
    a, b = F.Particles.from_numpy(w, s), F.Particles(n, torch.float32, True)
    src = torch.from_numpy(off0).cuda()
    want = np.argsort(s["key"], kind="stable")
    offs = np.concatenate([[0], np.cumsum(counts)])
    for rep in range(2):
        for sort in ("bin", "rebin"):
            off = torch.full((nc + 1,), -7, dtype=torch.int32, device="cuda")
            perm = torch.full((n,), -7, dtype=torch.int32, device="cuda")
            if sort == "bin":
                ctx.bin(a, b, off, perm)
            else:
                ctx.rebin(a, src, b, off, perm)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(off.cpu().numpy(), offs)
            np.testing.assert_array_equal(perm.cpu().numpy(), want)
            np.testing.assert_array_equal(b.numpy()["vx"], s["vx"][want])
    assert ctx.error_count() == 0
