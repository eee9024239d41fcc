"""GPU tests of the interpolation systems (k = 3, 4, 5) as padding values and
stored symbols: lines shorter than, equal to and longer than the reach of the
padding values' coefficients (24, 32, 42 entries), in both directions, on
noise (every frequency present), forward and adjoint against the oracle.  The
bars are those of the two precisions: 1e-12 and 1e-6 of the largest value."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

SIZES = [(4, 48), (24, 16), (12, 96), (64, 32), (48, 8), (128, 4)]


@pytest.mark.parametrize("k", [3, 4, 5])
@pytest.mark.parametrize("nx,ny", SIZES, ids=[f"{a}x{b}" for a, b in SIZES])
def test_noise_forward_and_adjoint(nx, ny, k):
    import torch
    import paper_1904_07400_amd as sg
    dom = (-1.0, 1.0, -0.5, 0.5)
    rng = np.random.default_rng(100 * k + nx)
    s, gx, gy = (rng.standard_normal((ny, nx)).astype(np.float32).astype(np.float64) for _ in range(3))
    rx, ry = oracle.forces(s, k, dom)
    rg = oracle.forces_adjoint(gx, gy, k, dom)
    for prec, tol in ((sg.SG_FP64, 1e-12), (sg.SG_FP32_SPLIT, 1e-6)):
        plan = sg.Plan([(nx, ny, *dom, k)], prec)
        try:
            fx, fy = plan.forces(to_dev(s.ravel(), plan.dtype))
            g = plan.adjoint(to_dev(gx.ravel(), plan.dtype), to_dev(gy.ravel(), plan.dtype))
            torch.cuda.synchronize()
            fx, fy, g = (v.double().cpu().numpy().reshape(ny, nx) for v in (fx, fy, g))
        finally:
            plan.close()
        scale = max(np.abs(rx).max(), np.abs(ry).max())
        assert max(np.abs(fx - rx).max(), np.abs(fy - ry).max()) <= tol * scale, (prec, "forces")
        assert np.abs(g - rg).max() <= tol * np.abs(rg).max(), (prec, "adjoint")
