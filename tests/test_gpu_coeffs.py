"""GPU tests of the written-out spline coefficients on both sides of the column
solve's line (1024 rows; from there on chunks of 32 rows with margins, tiles of 64
columns) and in place, on noise against the oracle.  Bars: 1e-13 of the largest
value (FP64; the systems amplify by at most 23), 1e-6 for single floats (two
roundings of 6e-8, the first amplified by at most 4.8)."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

SIZES = [(4, 4), (64, 64), (48, 768), (4, 1024), (96, 1024), (64, 1536), (24, 2048), (192, 2048)]


@pytest.mark.parametrize("k", [3, 4, 5])
@pytest.mark.parametrize("nx,ny", SIZES, ids=[f"{a}x{b}" for a, b in SIZES])
def test_chunked_column_solve(nx, ny, k):
    import torch
    import paper_1904_07400_amd as sg
    rng = np.random.default_rng(31 * k + nx + ny)
    s = rng.standard_normal((ny, nx)).astype(np.float32).astype(np.float64)
    ref = oracle.bspline_coeffs(s, k)
    for prec, tol in ((sg.SG_FP64, 1e-13), (sg.SG_FP32_SPLIT, 1e-6)):
        plan = sg.Plan([(nx, ny, -1.0, 1.0, -0.5, 0.5, k)], prec)
        try:
            x = to_dev(s.ravel(), plan.dtype)
            out = plan.coeffs(x)
            plan.coeffs(x, x)  # in place
            torch.cuda.synchronize()
            assert torch.equal(out, x), prec
            c = out.double().cpu().numpy().reshape(ny, nx)
        finally:
            plan.close()
        assert np.abs(c - ref).max() <= tol * np.abs(ref).max(), prec
