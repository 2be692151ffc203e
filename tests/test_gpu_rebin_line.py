"""The re-sort at the cell counts around the line between its narrow and wide count workgroups
(204,800 lanes: 3200 cells at 64 lanes, 6400 at 32) and where the grid ends inside a
workgroup, against the stable counting sort, as in the general test."""
import numpy as np
import pytest

from paper_2606_15622_amd import inputs as I
from test_gpu_rebin import fp, run_rebin
from test_gpu_rebin_sizes import state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,lanes", [(457, 7, 64), (50, 64, 64), (97, 33, 64), (6399, 1, 32), (80, 80, 32)])
@pytest.mark.parametrize("far", [0, 300])
def test_cell_counts_around_the_count_workgroups(nx, ny, lanes, far):
    F = fp()
    rng = np.random.default_rng(nx + far)
    w = I.cavity(ncell=8, ppc=4, precision="f32")
    w = dict(w, nx=nx, ny=ny, lx=nx * w["dx"], ly=ny * w["dy"], lanes=lanes)
    s, off0 = state(w, rng.integers(0, 12, nx * ny), rng, far)
    run_rebin(F, w, s, off0)
