"""CPU emulation of the 16-element column kernel (paper_1904_07400_amd/csrc/
colw.hpp) under ThreadSanitizer, against the column pass written from its
definition in numpy: every length, order and table form that the library
launches it with, on a few columns each (the packed column 0 among them)."""
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

GXX = shutil.which("g++")
pytestmark = [pytest.mark.slow, pytest.mark.skipif(GXX is None, reason="g++ not found")]

CASES = [(N, k, to) for N in (4096, 2048) for k, to in ((1, "float"), (2, "float2"), (3, "float"), (4, "float"),
                                                        (5, "float2"))]
CASES += [(1024, 1, "float2"), (1024, 4, "float2"), (512, 2, "float2"), (512, 3, "float2"), (256, 5, "float2"),
          (256, 2, "float2")]


def _build(tmp_path, N, k, to, adj):
    exe = str(tmp_path / "emu")
    r = subprocess.run([GXX, "-std=c++20", "-O1", "-g", "-fsanitize=thread", "-I" + os.path.join(HERE, "emu"),
                        "-I" + os.path.join(ROOT, "paper_1904_07400_amd", "csrc"), "-I" + os.path.join(ROOT, "include"),
                        f"-DEMU_TO={to}", f"-DEMU_N={N}", f"-DEMU_KIND={1 - k % 2}",
                        f"-DEMU_ORD={k if k >= 3 else 0}", f"-DEMU_ADJ={adj}",
                        os.path.join(HERE, "emu", "colw_driver.cpp"), "-o", exe, "-lpthread"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def _symbol(k, N):
    """The interpolation system's symbol along y, in the stored row's order (q even, then odd)."""
    st = cr.STENCIL[k]
    c = np.cos(np.pi * np.arange(2 * N) / N)
    sym = (st[len(st) // 2] + 2 * st[len(st) // 2 - 1] * c + (2 * (2 * c * c - 1) if k == 5 else 0)) / sum(st)
    return np.concatenate([sym[0:N + 1:2], sym[1:N:2]])


def _padding(k, N):
    """The padding values' coefficients c0, c1 (48 each) of order k's system on lines of N values."""
    bc = np.zeros((2, 48))
    if k >= 3:
        st, n = cr.STENCIL[k], min(N, 300)
        h, m = len(st) // 2, {3: 24, 4: 32, 5: 42}[k]
        G = np.linalg.inv(sum(np.diag([st[h + d]] * (n - abs(d)), d) for d in range(-h, h + 1)))
        bc[0, :m] = 76 * G[0, :m] + G[1, :m] if k == 5 else G[0, :m]
        bc[1, :m] = G[0, :m] if k == 5 else 0
    return bc


@pytest.mark.parametrize("N,k,to", CASES, ids=[f"{c[0]}-k{c[1]}-{c[2]}" for c in CASES])
def test_column_pass(tmp_path, N, k, to):
    exe = _build(tmp_path, N, k, to, 0)
    M = 4
    rng = np.random.default_rng(k * 17 + N)
    X = rng.standard_normal((M, N)) + 1j * rng.standard_normal((M, N))
    tx, ty, stored = fs._tables(rng, M, N, to)
    if k >= 3:  # the kernel's tables hold the system's symbol along y; the reference solves the system
        tx, ty = (t * _symbol(k, N) for t in (tx, ty))
    bc = _padding(k, N)
    xb = np.stack([X[:, ::-1][:, :48] @ bc[0], X[:, ::-1][:, :48] @ bc[1], X[:, :48] @ bc[0], X[:, :48] @ bc[1]], 1)
    fin, fout = str(tmp_path / "in.bin"), str(tmp_path / "out.bin")
    with open(fin, "wb") as f:
        X.astype(np.complex64).tofile(f)
        for t in stored:
            t.tofile(f)
        np.exp(-1j * np.pi * np.arange(2 * N) / N).astype(np.complex64).tofile(f)
        xb.astype(np.complex64).tofile(f)
    races = fs._run(exe, M, fin, fout)
    tj = int(np.fromfile(fout, dtype=np.int32, count=1)[0])
    V = cr.untile(np.fromfile(fout, dtype=np.complex64, offset=4), M, N, tj)
    ref = cr.column_pass(X.astype(np.complex64).astype(complex), tx, ty, k, M, N)
    assert races == 0
    assert np.abs(V - ref).max() / np.abs(ref).max() <= 1e-6


ADJ = [(4096, 1, "float"), (4096, 2, "float"), (4096, 3, "float2"), (4096, 4, "float"), (4096, 5, "float"),
       (2048, 3, "float"), (1024, 4, "float2")]


@pytest.mark.parametrize("N,k,to", ADJ, ids=[f"{c[0]}-k{c[1]}-{c[2]}" for c in ADJ])
def test_adjoint_column_pass(tmp_path, N, k, to):
    exe = _build(tmp_path, N, k, to, 1)
    M = 4
    rng = np.random.default_rng(k * 19 + N)
    Xx, Xy = (rng.standard_normal((M, N)) + 1j * rng.standard_normal((M, N)) for _ in range(2))
    tx, ty, stored = fs._tables(rng, M, N, to)
    if k >= 3:  # the kernel's tables hold the symbol; the reference solves the system
        tx, ty = (t * _symbol(k, N) for t in (tx, ty))
    fin, fout = str(tmp_path / "in.bin"), str(tmp_path / "out.bin")
    with open(fin, "wb") as f:
        Xx.astype(np.complex64).tofile(f)
        Xy.astype(np.complex64).tofile(f)
        for t in stored:
            t.tofile(f)
        np.exp(-1j * np.pi * np.arange(2 * N) / N).astype(np.complex64).tofile(f)
        _padding(k, N).tofile(f)
    races = fs._run(exe, M, fin, fout)
    tj = int(np.fromfile(fout, dtype=np.int32, count=1)[0])
    Y = cr.untile_half(np.fromfile(fout, dtype=np.complex64, offset=4), M, N, tj)
    ref = cr.adjoint_column_pass(Xx.astype(np.complex64).astype(complex), Xy.astype(np.complex64).astype(complex),
                                 tx, ty, k, M, N)
    assert races == 0
    assert np.abs(Y - ref).max() / np.abs(ref).max() <= 1e-6
