"""GPU test of the adjoint's last pass over every FP32 row length, whose rows share
a workgroup in slots spaced by the row length (lane by lane from four threads per
row on), with row counts that leave the last workgroup part empty: noise against
the oracle, 1e-6 of the largest value."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

LENGTHS = [4, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024, 1536, 2048, 4096, 8192]


@pytest.mark.parametrize("k,ny", [(1, 12), (3, 24)])
@pytest.mark.parametrize("nx", LENGTHS)
def test_adjoint_rows(nx, ny, k):
    import torch
    import paper_1904_07400_amd as sg
    dom = (-1.0, 1.0, -ny / nx, ny / nx)
    rng = np.random.default_rng(nx + k)
    gx, gy = (rng.standard_normal((ny, nx)).astype(np.float32).astype(np.float64) for _ in range(2))
    ref = oracle.forces_adjoint(gx, gy, k, dom)
    plan = sg.Plan([(nx, ny, *dom, k)], sg.SG_FP32_SPLIT)
    try:
        g = plan.adjoint(to_dev(gx.ravel(), plan.dtype), to_dev(gy.ravel(), plan.dtype))
        torch.cuda.synchronize()
        g = g.double().cpu().numpy().reshape(ny, nx)
    finally:
        plan.close()
    assert np.abs(g - ref).max() <= 1e-6 * np.abs(ref).max()
