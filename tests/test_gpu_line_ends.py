"""GPU tests of the padding values (k >= 3) at the ends of rows and columns, which
the lanes that hold those ends sum together: lengths with one, two, ... and all 32
of these lanes, shorter and longer than the coefficients' reach, in every form of
the forward row pass, and columns on both sides of the line (threads of one wave)
beyond which the row pass leaves them in parts; on noise against the oracle.
Bars: those of the two precisions, 1e-12 and 1e-6 of the largest value."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

SIZES = [(8, 8), (16, 12), (32, 8), (96, 4), (192, 8), (256, 12), (512, 8), (768, 16), (1024, 8), (1536, 4), (4096, 4),
         (8192, 8),
         (8, 16), (12, 24), (4, 64), (8, 128), (8, 192), (16, 256), (12, 384), (8, 512), (4, 768), (8, 1024),
         (12, 1536)]


@pytest.mark.parametrize("k", [3, 4, 5])
@pytest.mark.parametrize("nx,ny", SIZES, ids=[f"{a}x{b}" for a, b in SIZES])
def test_noise_to_the_ends_of_the_lines(nx, ny, k):
    import torch
    import paper_1904_07400_amd as sg
    dom = (-1.0, 1.0, -ny / nx, ny / nx)  # square cells
    s = np.random.default_rng(7 * k + nx).standard_normal((ny, nx)).astype(np.float32).astype(np.float64)
    rx, ry = oracle.forces(s, k, dom)
    scale = max(np.abs(rx).max(), np.abs(ry).max())
    for prec, tol in ((sg.SG_FP64, 1e-12), (sg.SG_FP32_SPLIT, 1e-6)):
        plan = sg.Plan([(nx, ny, *dom, k)], prec)
        try:
            fx, fy = plan.forces(to_dev(s.ravel(), plan.dtype))
            torch.cuda.synchronize()
            fx, fy = (v.double().cpu().numpy().reshape(ny, nx) for v in (fx, fy))
        finally:
            plan.close()
        assert max(np.abs(fx - rx).max(), np.abs(fy - ry).max()) <= tol * scale, prec
