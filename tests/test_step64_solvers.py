"""The FP64 step's 3x3 and 6x6 solvers on the CPU, against numpy: the solution of positive
definite systems, and no finite value for a system that is not positive definite (a diverged
sample's, made indefinite by its rounding), whichever pivot shows it: such a sample's state has
to be non-finite, for its cost to be +inf."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ is not available")
    so = str(tmp_path_factory.mktemp("step64") / "solvers.so")
    cs = os.path.join(ROOT, "paper_2409_10469_amd", "csrc")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wno-unknown-pragmas", "-Wno-attributes",
                        "-I", os.path.join(ROOT, "tests", "hostcheck"), "-I", cs, "-I", os.path.join(ROOT, "include"),
                        os.path.join(ROOT, "tests", "step64check", "solvers.cpp"), "-o", so],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return C.CDLL(so)


def _system(rng, pivots):
    """L diag(pivots) L^T with a unit lower L: a system with these pivots."""
    n = len(pivots)
    L = np.eye(n) + np.tril(rng.uniform(-0.5, 0.5, (n, n)), -1)
    A = L @ np.diag(pivots) @ L.T
    return (A + A.T) / 2


def _solve(lib, A, B):
    """The columns of A^-1 B by the library's solver of A's size."""
    n = len(A)
    dp = lambda a: a.ctypes.data_as(C.POINTER(C.c_double))
    if n == 3:
        a, b = np.ascontiguousarray(A[np.tril_indices(3)]), np.ascontiguousarray(B.T)
        lib.solve_3x3(dp(a), dp(b), C.c_int(B.shape[1]))
        return b.T
    out = np.empty_like(B)
    for j in range(B.shape[1]):
        q, r = np.ascontiguousarray(A[np.triu_indices(6)]), np.ascontiguousarray(B[:, j])
        lib.solve_6x6(dp(q), dp(r))
        out[:, j] = r
    return out


@pytest.mark.parametrize("n", [3, 6])
def test_positive_definite_systems(lib, n):
    rng = np.random.default_rng(n)
    for _ in range(50):
        A = _system(rng, 10.0 ** rng.uniform(-3, 3, n))
        B = rng.normal(size=(n, 4))
        x = _solve(lib, A, B)
        # forward error of a backward stable solve: kappa (n + 1) eps, twice for the assembly
        bound = 4 * (n + 1) * np.finfo(float).eps * np.linalg.cond(A) * np.abs(np.linalg.solve(A, B)).max()
        assert np.abs(x - np.linalg.solve(A, B)).max() <= bound


@pytest.mark.parametrize("pivot", [-1.0, -1e-3, -1e6, 0.0, -1e150, float("nan")])
@pytest.mark.parametrize("n", [3, 6])
def test_systems_without_a_cholesky_factor_give_no_finite_value(lib, n, pivot):
    rng = np.random.default_rng(10 + n)
    for at in range(n):
        d = 10.0 ** rng.uniform(-1, 1, n)
        d[at] = 1.0
        A = _system(rng, d)
        # the last pivot that this entry forms, moved to the wanted value: pivots before it stay
        A[at, at] = A[at, at] - 1.0 + pivot
        if pivot == 0.0 and at:
            A[at, :at] = A[:at, at] = 0.0
            A[at, at] = 0.0
        x = _solve(lib, A, rng.normal(size=(n, 3)))
        assert not np.isfinite(x).any(), (at, x)
