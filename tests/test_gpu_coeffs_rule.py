"""GPU tests of the written-out coefficients on both sides of the rule that picks
the column solve by the grid's size and order (whole columns in place, or chunks
by way of the spectra buffer): out of place, in place and, after a force step on
the same plan, again, on noise against the oracle.  Bars: 1e-13 of the largest
value (FP64; the systems amplify by at most 23), 1e-6 for single floats (two
roundings of 6e-8, the first amplified by at most 4.8)."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

# k = 3, 4 change at 2^18 cells, at 2^17 from 2048 rows and at 8192 rows; k = 5 at 2^19 cells
SIZES = [(192, 1024), (256, 1024), (512, 1024), (48, 2048), (64, 2048), (256, 2048), (4, 4096), (32, 4096), (4, 8192),
         (64, 8192)]


@pytest.mark.parametrize("k", [3, 4, 5])
@pytest.mark.parametrize("nx,ny", SIZES, ids=[f"{a}x{b}" for a, b in SIZES])
def test_column_solve_by_size(nx, ny, k):
    import torch
    import paper_1904_07400_amd as sg
    rng = np.random.default_rng(17 * k + nx + ny)
    s = rng.standard_normal((ny, nx)).astype(np.float32).astype(np.float64)
    ref = oracle.bspline_coeffs(s, k)
    for prec, tol in ((sg.SG_FP64, 1e-13), (sg.SG_FP32_SPLIT, 1e-6)):
        plan = sg.Plan([(nx, ny, -1.0, 1.0, -ny / nx, ny / nx, k)], prec)  # square cells: a quick plan
        try:
            x = to_dev(s.ravel(), plan.dtype)
            out = plan.coeffs(x)
            plan.forces(x)
            again = plan.coeffs(x)
            plan.coeffs(x, x)  # in place
            torch.cuda.synchronize()
            assert torch.equal(out, x) and torch.equal(out, again), prec
            c = out.double().cpu().numpy().reshape(ny, nx)
        finally:
            plan.close()
        assert np.abs(c - ref).max() <= tol * np.abs(ref).max(), prec
