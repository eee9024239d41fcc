"""CPU emulation, under ThreadSanitizer, of the column kernels in the forms that the
library launches: the interpolation systems of k >= 3 in the tables, their padding
values read as several parts each (forward) or added at the columns' ends
(adjoint), columns of 8192 from column-major and from tiled row spectra, and the
plan-time spectrum columns with the systems' symbols.  Reference: the column
pass written from its definition in numpy, the systems solved.  Bars: 1e-6 (FP32)
and 1e-13 (FP64) of the largest value."""
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
sys.path.insert(0, os.path.join(HERE, "emu"))
sys.path.insert(0, HERE)
import colpass_ref as cr  # noqa: E402
import test_emu_colfs as fs  # noqa: E402
import test_emu_colw as cw  # noqa: E402

GXX = shutil.which("g++")
pytestmark = [pytest.mark.slow, pytest.mark.skipif(GXX is None, reason="g++ not found")]

COLFS, COLFS_XY, COLFS3, COLW, COLFS_ADJ, SPECFS = range(6)


def _build(tmp_path, kernel, prec, to, N, E, slots, k, split=0, xt=0, pg=1):
    exe = str(tmp_path / "emu")
    r = subprocess.run([GXX, "-std=c++20", "-O1", "-g", "-fsanitize=thread", "-I" + os.path.join(HERE, "emu"),
                        "-I" + os.path.join(ROOT, "paper_1904_07400_amd", "csrc"), "-I" + os.path.join(ROOT, "include"),
                        f"-DEMU_KERNEL={kernel}", f"-DEMU_R={'float' if prec == 32 else 'double'}", f"-DEMU_TO={to}",
                        f"-DEMU_N={N}", f"-DEMU_E={E}", f"-DEMU_SLOTS={slots}", f"-DEMU_SPLIT={split}",
                        f"-DEMU_KIND={1 - k % 2}", f"-DEMU_ORD={k if k >= 3 else 0}", f"-DEMU_XT={xt}", f"-DEMU_PG={pg}",
                        os.path.join(HERE, "emu", "colpad_driver.cpp"), "-o", exe, "-lpthread"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def _tiled(X):
    """Bin p of row j at x_base(p) + x_at(j): tiles of two bins of one parity by four rows."""
    M, N = X.shape
    out = np.empty(M * N, X.dtype)
    j = np.arange(N)
    for p in range(M):
        q = p >> 1
        out[((p & 1) * (M // 2) + (q & ~1)) * N + (q & 1) * 4 + (j >> 2) * 8 + (j & 3)] = X[p]
    return out


def _parts(rng, X, k, N, pg, cdt):
    """The padding values of slots N, N + 1, -1, -2 of every column, each split into pg parts: [part][column][slot]."""
    bc = cw._padding(k, N)
    v = np.stack([X[:, ::-1][:, :48] @ bc[0], X[:, ::-1][:, :48] @ bc[1], X[:, :48] @ bc[0], X[:, :48] @ bc[1]], 1)
    out = 0.1 * (rng.standard_normal((pg, *v.shape)) + 1j * rng.standard_normal((pg, *v.shape)))
    out[-1] = v - out[:-1].sum(0)
    return out.astype(cdt)


# kernel, precision, tables, N, E, LDS slots, order, component split, tiled, parts
FWD = [(COLFS, 64, "double", 1024, 8, 2, 4, 0, 0, 3), (COLFS, 64, "double", 2048, 8, 2, 5, 0, 0, 42),
       (COLFS, 64, "double", 8192, 16, 1, 4, 1, 0, 16), (COLFS, 32, "float", 2048, 8, 2, 3, 0, 0, 6),
       (COLFS, 32, "float2", 2048, 8, 2, 4, 0, 0, 8), (COLFS_XY, 32, "float", 8192, 16, 2, 3, 0, 1, 6),
       (COLFS_XY, 32, "float2", 8192, 16, 2, 4, 0, 1, 8), (COLFS_XY, 32, "float", 8192, 16, 2, 5, 0, 0, 11),
       (COLFS3, 32, "float2", 1536, 8, 4, 4, 0, 0, 8), (COLFS3, 32, "float2", 768, 4, 4, 5, 0, 0, 11),
       (COLW, 32, "float", 4096, 16, 2, 4, 0, 0, 8), (COLW, 32, "float2", 4096, 16, 2, 1, 0, 0, 1),
       (COLW, 32, "float2", 4096, 16, 2, 3, 0, 0, 6)]


@pytest.mark.parametrize("kernel,prec,to,N,E,slots,k,split,xt,pg", FWD,
                         ids=[f"{c[0]}-fp{c[1]}-{c[3]}-k{c[6]}-{c[2]}-xt{c[8]}-{c[9]}parts" for c in FWD])
def test_column_pass(tmp_path, kernel, prec, to, N, E, slots, k, split, xt, pg):
    exe = _build(tmp_path, kernel, prec, to, N, E, slots, k, split, xt, pg)
    M, cdt = 4, np.complex64 if prec == 32 else np.complex128
    rng = np.random.default_rng(k * 23 + N + kernel)
    X = (rng.standard_normal((M, N)) + 1j * rng.standard_normal((M, N))).astype(cdt)
    tx, ty, stored = fs._tables(rng, M, N, to)
    if k >= 3:  # the kernel's tables hold the symbol along y; the reference solves the system
        tx, ty = (t * cw._symbol(k, N) for t in (tx, ty))
    fin, fout = str(tmp_path / "in.bin"), str(tmp_path / "out.bin")
    with open(fin, "wb") as f:
        (_tiled(X) if xt else X).tofile(f)
        for t in stored:
            t.tofile(f)
        np.exp(-1j * np.pi * np.arange(2 * N) / N).astype(cdt).tofile(f)
        _parts(rng, X, k, N, pg, cdt).tofile(f)
    races = fs._run(exe, M, fin, fout)
    tj = int(np.fromfile(fout, dtype=np.int32, count=1)[0])
    V = cr.untile(np.fromfile(fout, dtype=cdt, offset=4), M, N, tj)
    ref = cr.column_pass(X.astype(complex), tx, ty, k, M, N)
    assert races == 0
    assert np.abs(V - ref).max() / np.abs(ref).max() <= (1e-6 if prec == 32 else 1e-13)


ADJ = [(64, "double", 1024, 8, 2, 4, 0), (64, "double", 8192, 16, 1, 3, 0), (32, "float", 2048, 8, 2, 5, 0),
       (32, "float", 8192, 16, 2, 3, 1), (32, "float2", 8192, 16, 2, 4, 1), (32, "float", 8192, 16, 2, 5, 0)]


@pytest.mark.parametrize("prec,to,N,E,slots,k,xt", ADJ, ids=[f"fp{c[0]}-{c[2]}-k{c[5]}-{c[1]}-xt{c[6]}" for c in ADJ])
def test_adjoint_column_pass(tmp_path, prec, to, N, E, slots, k, xt):
    exe = _build(tmp_path, COLFS_ADJ, prec, to, N, E, slots, k, 0, xt)
    M, cdt = 4, np.complex64 if prec == 32 else np.complex128
    rng = np.random.default_rng(k * 29 + N)
    Xx, Xy = ((rng.standard_normal((M, N)) + 1j * rng.standard_normal((M, N))).astype(cdt) for _ in range(2))
    tx, ty, stored = fs._tables(rng, M, N, to)
    if k >= 3:
        tx, ty = (t * cw._symbol(k, N) for t in (tx, ty))
    fin, fout = str(tmp_path / "in.bin"), str(tmp_path / "out.bin")
    with open(fin, "wb") as f:
        for X in (Xx, Xy):
            (_tiled(X) if xt else X).tofile(f)
        for t in stored:
            t.tofile(f)
        np.exp(-1j * np.pi * np.arange(2 * N) / N).astype(cdt).tofile(f)
        cw._padding(k, N).tofile(f)
    races = fs._run(exe, M, fin, fout)
    tj = int(np.fromfile(fout, dtype=np.int32, count=1)[0])
    Y = cr.untile_half(np.fromfile(fout, dtype=cdt, offset=4), M, N, tj)
    ref = cr.adjoint_column_pass(Xx.astype(complex), Xy.astype(complex), tx, ty, k, M, N)
    assert races == 0
    assert np.abs(Y - ref).max() / np.abs(ref).max() <= (1e-6 if prec == 32 else 1e-13)


@pytest.mark.parametrize("k,to", [(4, "double"), (5, "float2")])
def test_spectrum_columns_with_symbols(tmp_path, k, to):
    M, N = 4, 8192
    exe = _build(tmp_path, SPECFS, 64, to, N, 16, 1, k)
    rng = np.random.default_rng(k + 5)
    Sg = rng.standard_normal((M, 2 * N)) + 1j * rng.standard_normal((M, 2 * N))
    fin, fout = str(tmp_path / "in.bin"), str(tmp_path / "out.bin")
    with open(fin, "wb") as f:
        Sg.tofile(f)
        np.exp(-1j * np.pi * np.arange(2 * N) / N).tofile(f)
    races = fs._run(exe, M, fin, fout)
    raw = np.fromfile(fout, dtype=np.float64 if to == "double" else np.float32, offset=4)
    got = raw.reshape(M + 1, N + 1, 2).astype(np.float64).sum(-1) if to == "float2" else \
        raw.reshape(M + 1, N + 1).astype(np.float64)
    sx = cw._symbol(k, M)  # bins 0, 2, .. M, then 1, 3, ..
    symx = np.empty(M + 1)
    symx[0::2], symx[1::2] = sx[:M // 2 + 1], sx[M // 2 + 1:]
    ref = cr.spectrum_columns(Sg, k, M, N, 0.25) / symx[:, None] / cw._symbol(k, N)[None, :]
    assert races == 0
    assert np.abs(got - ref).max() / np.abs(ref).max() <= (1e-7 if to == "float" else 1e-13)
