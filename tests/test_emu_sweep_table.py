"""CPU check of the one-launch kernels' coefficient table (build_sweep_table):
tests/emu/sweep_table_emu.cpp replays a solve on it, and the result must equal
LAPACK's for every matrix kind, direction and chunk size, for full
decompositions (periodic correction in the chunks' boundary states) and
ragged ones (correction rows; the last real chunk ending at row n - 1, with
one row or many)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2107_05395_amd import inputs

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2107_05395_amd", "csrc")
SRC = os.path.join(HERE, "emu", "sweep_table_emu.cpp")
LIB = os.path.join(HERE, "emu", "libsweep_table_emu.so")


@pytest.fixture(scope="module")
def emu():
    deps = [SRC] + [os.path.join(CSRC, p) for p in ("factor.cpp", "factor.h", "internal.h")]
    if not os.path.exists(LIB) or os.path.getmtime(LIB) < max(map(os.path.getmtime, deps)):
        tmp = LIB + ".tmp%d" % os.getpid()
        subprocess.run(["/opt/rocm/bin/hipcc", "-O1", "-std=c++17", "-fPIC", "-shared", SRC, deps[1],
                        "-o", tmp], check=True)
        os.replace(tmp, LIB)
    lib = ctypes.CDLL(LIB)
    P = ctypes.POINTER(ctypes.c_double)
    lib.emu_sweep.argtypes = [ctypes.c_int] + [P] * 5 + [ctypes.c_int64, ctypes.c_int, ctypes.c_int, P, P]
    return lib


CASES = [(n, C) for n in (4, 5, 8, 16, 17, 33, 64, 65, 66, 128, 129, 256, 257, 500, 512, 1000, 1024)
         for C in (4, 8, 16, 32, 64, 128) if (n + C - 1) // C <= 64]


@pytest.mark.parametrize("kind", ["tri", "tri_cyclic", "penta", "penta_cyclic"])
@pytest.mark.parametrize("adjoint", [0, 1])
def test_solve_on_the_sweep_table(emu, kind, adjoint):
    kid = ["tri", "tri_cyclic", "penta", "penta_cyclic"].index(kind)
    P = ctypes.POINTER(ctypes.c_double)
    for n, C in CASES:
        if kind == "penta_cyclic" and n < 5:
            continue
        bands = (inputs.random_dominant_tri if kind.startswith("tri") else inputs.random_dominant_penta)(n, n + C)
        f = inputs.uniform_batch(n, 1, seed=n + C)
        arrs = [np.ascontiguousarray(b) for b in bands] + [np.zeros(n)] * (5 - len(bands))
        x = np.empty(n)
        rhs = np.ascontiguousarray(f[:, 0])
        assert emu.emu_sweep(kid, *(b.ctypes.data_as(P) for b in arrs), n, adjoint, C,
                             rhs.ctypes.data_as(P), x.ctypes.data_as(P)) == 0
        K, A = len(bands) // 2, np.zeros((n, n))
        for q, b in enumerate(bands):
            for i in range(n):
                j = i + q - K
                if 0 <= j < n or kind.endswith("cyclic"):
                    A[i, j % n] += b[i]
        ref = np.linalg.solve(A.T if adjoint else A, rhs)
        # backward-stable solves of a matrix with condition kappa: 2 kappa u
        tol = max(1e-13, 4.0 * np.linalg.cond(A) * 2.0 ** -53)
        assert np.linalg.norm(x - ref) <= tol * np.linalg.norm(ref), (n, C)
