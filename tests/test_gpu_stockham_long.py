"""GPU test of the Stockham column kernels at the lengths that the four-step pass
takes otherwise (SG_COLFS=0, a diagnostic): forward and adjoint against the oracle.
Their FP64 columns of 4096 need more than 64 KB of LDS, which every kernel sized at
launch has to ask for.  Bars: 1e-12 and 1e-6 of the largest value."""
import ctypes
import os
import re

import numpy as np
import pytest

import oracle
from gpu_util import to_dev

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1904_07400_amd", "csrc",
                   "sg_kernels.hip")


def test_every_kernel_sized_at_launch_asks_for_its_lds():
    src = open(SRC).read()
    kernels = set()
    for body in re.split(r"\n__global__ ", src)[1:]:
        name = re.search(r"\b(k_\w+)\(", body).group(1)
        if "extern __shared__" in body.split("\n}\n")[0]:
            kernels.add(name)
    assert {"k_row_fwd", "k_col", "k_col_adj", "k_row_inv", "k_row_c2r"} <= kernels
    for k in kernels:
        assert re.search(r"dyn_lds_optin<&" + k + "<", src), k


@pytest.mark.gpu
@pytest.mark.parametrize("k", [1, 2, 3, 5])
@pytest.mark.parametrize("nx,ny", [(8, 1024), (16, 1536), (8, 2048), (8, 4096)], ids=["1024", "1536", "2048", "4096"])
def test_long_columns(nx, ny, k, monkeypatch):
    import torch
    import paper_1904_07400_amd as sg
    monkeypatch.setenv("SG_COLFS", "0")
    libc = ctypes.CDLL(None)
    libc.getenv.restype = ctypes.c_char_p
    assert libc.getenv(b"SG_COLFS") == b"0"
    dom = (-1.0, 1.0, -ny / nx, ny / nx)
    rng = np.random.default_rng(ny + k)
    s, gx, gy = (rng.standard_normal((ny, nx)).astype(np.float32).astype(np.float64) for _ in range(3))
    rx, ry = oracle.forces(s, k, dom)
    rg = oracle.forces_adjoint(gx, gy, k, dom)
    scale = max(np.abs(rx).max(), np.abs(ry).max())
    for prec, tol in ((sg.SG_FP64, 1e-12), (sg.SG_FP32_SPLIT, 1e-6)):
        plan = sg.Plan([(nx, ny, *dom, k)], prec)
        try:
            fx, fy = plan.forces(to_dev(s.ravel(), plan.dtype))
            g = plan.adjoint(to_dev(gx.ravel(), plan.dtype), to_dev(gy.ravel(), plan.dtype))
            torch.cuda.synchronize()
            fx, fy, g = (v.double().cpu().numpy().reshape(ny, nx) for v in (fx, fy, g))
        finally:
            plan.close()
        assert max(np.abs(fx - rx).max(), np.abs(fy - ry).max()) <= tol * scale, (prec, "forces")
        assert np.abs(g - rg).max() <= tol * np.abs(rg).max(), (prec, "adjoint")
