"""GPU test of the launch tiles alone: plans whose rows and columns per workgroup were
timed (SG_TUNE=quick times tiles and leaves the launch variants, which may round
otherwise) against plans with the launch rules' own, bit for bit, forward and
adjoint."""
import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(12, 96), (48, 48), (512, 24), (384, 768), (512, 1024), (1536, 96), (8192, 64)]


@pytest.mark.parametrize("k", [1, 4, 5])
@pytest.mark.parametrize("nx,ny", SHAPES, ids=[f"{a}x{b}" for a, b in SHAPES])
def test_timed_tiles_change_no_bit(nx, ny, k, monkeypatch):
    import torch
    import paper_1904_07400_amd as sg
    rng = np.random.default_rng(nx + 3 * ny + k)
    s, gx, gy = (rng.standard_normal(nx * ny) for _ in range(3))
    for prec in (sg.SG_FP64, sg.SG_FP32_SPLIT):
        def run(mode):
            if mode:
                monkeypatch.setenv("SG_TUNE", mode)
            else:
                monkeypatch.delenv("SG_TUNE", raising=False)
            plan = sg.Plan([(nx, ny, -1.0, 1.0, -ny / nx, ny / nx, k)], prec)
            try:
                fx, fy = plan.forces(to_dev(s, plan.dtype))
                g = plan.adjoint(to_dev(gx, plan.dtype), to_dev(gy, plan.dtype))
                torch.cuda.synchronize()
                return sg.sg_plan_tuning(plan.handle, 0), [v.cpu().numpy() for v in (fx, fy, g)]
            finally:
                plan.close()
        t0, one = run(None)
        t1, other = run("quick")
        assert t0[0] == t1[0], "the launch variants are the same"
        for v, w in zip(one, other):
            assert np.isfinite(v).all() and np.array_equal(v, w), prec
