"""GPU tests of the launch rules: the rows and columns per workgroup that a plan's
default launch takes depend on the number of grids in the class, and a result must
not (bit-identical: every line's arithmetic, and the grouping of the padding
values' parts, is that of the line length).  One grid against the same grid as the
first and last of a class large enough to move every rule, and against a plan with
timed tiles, forward and adjoint."""
import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu

# nx, ny, grids in the class
SHAPES = [(4, 4, 40), (32, 32, 40), (12, 96, 24), (512, 24, 24), (256, 256, 9), (768, 384, 6), (384, 768, 6),
          (512, 1024, 5), (1536, 96, 9)]


@pytest.mark.parametrize("k", [2, 3, 5])
@pytest.mark.parametrize("nx,ny,ng", SHAPES, ids=[f"{a}x{b}x{c}" for a, b, c in SHAPES])
def test_result_does_not_depend_on_the_launch(nx, ny, ng, k):
    import torch
    import paper_1904_07400_amd as sg
    dom = (-1.0, 1.0, -0.5, 0.5)
    rng = np.random.default_rng(nx + 7 * ny + k)
    s, gx, gy = (rng.standard_normal(nx * ny) for _ in range(3))
    for prec in (sg.SG_FP64, sg.SG_FP32_SPLIT):
        def run(n, flags=0):
            plan = sg.Plan([(nx, ny, *dom, k)] * n, prec, flags=flags)
            try:
                a, b, c = (to_dev(np.tile(v, n), plan.dtype) for v in (s, gx, gy))
                fx, fy = plan.forces(a)
                g = plan.adjoint(b, c)
                torch.cuda.synchronize()
                return [v.cpu().numpy().reshape(n, -1) for v in (fx, fy, g)]
            finally:
                plan.close()
        one = run(1)
        assert all(np.isfinite(v).all() and np.abs(v).max() > 0 for v in one)
        for other in (run(ng), run(1, sg.SG_FLAG_AUTOTUNE)):
            for v, w in zip(one, other):
                for row in (w[0], w[-1]):
                    assert np.array_equal(v[0], row), prec
