"""GPU test of what a non-finite density value does to the written-out coefficients,
on both sides of the rule that picks the column solve: the cells of its row and
column within the systems' reach (24, 32, 42 cells for k = 3, 4, 5) are
non-finite, those more than 96 cells away are finite and the same as without it."""
import pytest

pytestmark = pytest.mark.gpu

REACH = {3: 24, 4: 32, 5: 42}


@pytest.mark.parametrize("k", [3, 4, 5])
@pytest.mark.parametrize("nx,ny", [(256, 512), (256, 1024), (512, 2048)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_reach_of_a_non_finite_value(nx, ny, k, bad):
    import torch
    import paper_1904_07400_amd as sg
    for prec in (sg.SG_FP64, sg.SG_FP32_SPLIT):
        plan = sg.Plan([(nx, ny, -1.0, 1.0, -ny / nx, ny / nx, k)], prec)
        try:
            s = torch.rand(ny, nx, dtype=plan.dtype, device="cuda")
            ref = plan.coeffs(s.reshape(-1)).view(ny, nx).clone()
            for j, i in ((0, nx - 1), (ny // 2, nx // 2), (ny // 2 + 17, 5), (ny - 3, nx // 2 + 1)):
                x = s.clone()
                x[j, i] = bad
                c = plan.coeffs(x.reshape(-1)).view(ny, nx)
                jj = (torch.arange(ny, device="cuda") - j).abs()
                ii = (torch.arange(nx, device="cuda") - i).abs()
                assert not torch.isfinite(c[jj <= REACH[k], i]).any()
                assert not torch.isfinite(c[j, ii <= REACH[k]]).any()
                far = (jj[:, None] > 96) | (ii[None, :] > 96)
                assert torch.equal(c[far], ref[far])
        finally:
            plan.close()
