"""The one-kernel LITE closure of third-order records against the network kernel followed by the
check kernel, with NaN told from zero: update records hold no NaN whatever the cell's moments,
and the standardised outputs have one in both or in neither."""
import math

import pytest
import torch

from test_gpu_lite_sizes import fp, params, records, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [9, 129, 32769])
def test_records_are_finite_and_equal(n):
    F = fp()
    mom, pd = records(n, n + 1), params(6)
    prev = torch.full((n, 16), 1e5, dtype=torch.float64, device="cuda")
    prev[:, 14] = float(F.CELL_NN)
    for relax in (1.0, 0.3):
        rec, st = run(F, mom, 3, pd, relax, prev)
        rec5, st5 = run(F, mom, 5, pd, relax, prev)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(rec).all()) and torch.equal(rec, rec5) and torch.equal(st, st5)
    y = run(F, mom, 3, pd, 1.0, prev, outputs=True)
    last = run(F, mom[n - 5:].contiguous(), 3, pd, 1.0, prev, outputs=True)
    torch.cuda.synchronize()
    good = torch.isfinite(mom).all(1)
    assert bool(torch.isfinite(y[good]).all())
    assert torch.equal(y[n - 5:].isnan(), last.isnan()) and torch.equal(y[n - 5:].nan_to_num(), last.nan_to_num())
    assert math.isfinite(float(y[good].abs().max()))
