"""GPU parity of large grids with mass at their edges, where the padding values of the
interpolation systems (k >= 3) lie and workgroups loop over many columns: impulses
in the four corners and 1 to 41 cells from the edges (the coefficients reach 24,
32 and 42 cells), columns of every long kernel, against the oracle's exact
superposition around every impulse, along the edges and at sampled cells.  Bars:
1e-12 and 1e-6 of the largest value."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import run_forces

pytestmark = pytest.mark.gpu

# nx, ny, orders, FP64 as well
CASES = [(1024, 2048, k, True) for k in (3, 4, 5)] + [(2048, 1024, 3, True), (2048, 2048, 5, True)] + \
        [(4096, 4096, k, k == 3) for k in (3, 4, 5)] + [(8192, 4096, 4, False), (4096, 8192, 5, False)] + \
        [(8192, 8192, k, False) for k in (3, 4, 5)]


@pytest.mark.parametrize("M,N,k,f64", CASES, ids=[f"{c[0]}x{c[1]}-k{c[2]}" for c in CASES])
def test_impulses_at_the_edges(M, N, k, f64):
    import paper_1904_07400_amd as sg
    si = np.array([0, M - 1, 0, M - 1, 1, M - 3, 5, M - 8, 23, M - 32, 40, M - 42, M // 3, M // 2, 0, M - 1], np.int32)
    sj = np.array([0, 0, N - 1, N - 1, N - 2, 2, 7, N - 6, N - 24, 31, 41, N - 41, 0, N - 1, N // 3, N // 2], np.int32)
    sc = np.array([1, -.75, .5, .25, -.6, .8, -1, .9, .7, -.5, .6, -.9, .8, -.7, 1, -.4])
    C = np.zeros((N, M))
    np.add.at(C, (sj, si), sc)
    sigma = oracle.bspline_apply(C, k)
    del C
    near = {int(min(max(b + db, 0), N - 1)) * M + int(min(max(a + da, 0), M - 1))
            for a, b in zip(si, sj) for da in (-1, 0, 1) for db in (-1, 0, 1)}
    edge = {j * M + i for j in (0, N - 1) for i in range(0, M, 37)} | {j * M + i for j in range(0, N, 41) for i in (0, M - 1)}
    cells = workloads.sample_cells(31 + k, M, N, 100, extra=sorted(near | edge))
    rx, ry = oracle.forces_sparse(k, 2.0 / M, 2.0 / M, M, si, sj, sc, cells)
    scale = max(np.abs(rx).max(), np.abs(ry).max())
    half = N / M
    for prec, tol in ((sg.SG_FP64, 1e-12),) * f64 + ((sg.SG_FP32_SPLIT, 1e-6),):
        gx, gy = run_forces((M, N, -1.0, 1.0, -half, half, k), prec, sigma)
        err = max(np.abs(gx.ravel()[cells] - rx).max(), np.abs(gy.ravel()[cells] - ry).max()) / scale
        assert err <= tol, (prec, err)
