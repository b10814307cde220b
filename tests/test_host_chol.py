"""The free root's 6 x 6 Cholesky solve, whose quotients come from one
reciprocal per diagonal entry: the bits of the same solve with divisions."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2109_07719_amd", "csrc")
SOURCE = """
#include "%s/aba_lane.h"
template <typename S> void run(int n, const S* A, const S* b, S* x) {
  using namespace aba;
  for (; n-- > 0; A += 36, b += 6, x += 6) {
    auto sym = [&](int o) { return sy3<S>(A[7 * o], A[7 * o + 7], A[7 * o + 14], A[7 * o + 1], A[7 * o + 2], A[7 * o + 8]); };
    SySp<S> M;
    M.A = sym(0);
    M.C = sym(3);
    for (int i = 0; i < 3; ++i)
      for (int j = 0; j < 3; ++j) M.B.m[3 * i + j] = A[6 * i + 3 + j];
    const V6<S> r = chol6_solve(chol6(M), v6<S>(v3<S>(b[0], b[1], b[2]), v3<S>(b[3], b[4], b[5])));
    const S o[6] = {r.a.x, r.a.y, r.a.z, r.l.x, r.l.y, r.l.z};
    for (int k = 0; k < 6; ++k) x[k] = o[k];
  }
}
extern "C" void run_f(int n, const float* A, const float* b, float* x) { run(n, A, b, x); }
extern "C" void run_d(int n, const double* A, const double* b, double* x) { run(n, A, b, x); }
"""


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_quotients_are_the_divisions(tmp_path, dtype):
    src, so = tmp_path / "chol.cpp", tmp_path / "chol.so"
    src.write_text(SOURCE % os.path.abspath(CSRC))
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-Wno-unknown-pragmas",
                           "-o", str(so), str(src)])
    n, rng = 2000, np.random.default_rng(1)
    M = rng.normal(size=(n, 6, 6))
    A = (M @ M.transpose(0, 2, 1) + 0.1 * np.eye(6)).astype(dtype)
    A = np.ascontiguousarray(np.tril(A) + np.tril(A, -1).transpose(0, 2, 1))
    b = rng.normal(size=(n, 6)).astype(dtype)
    x = np.empty_like(b)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    getattr(ctypes.CDLL(str(so)), "run_f" if dtype == np.float32 else "run_d")(n, p(A), p(b), p(x))
    L, y = np.zeros_like(A), b.copy()
    for i in range(6):
        for j in range(i + 1):
            s = A[:, i, j]
            for k in range(j):
                s = s - L[:, i, k] * L[:, j, k]
            L[:, i, j] = np.sqrt(s) if i == j else s / L[:, j, j]
    for i in range(6):
        for k in range(i):
            y[:, i] = y[:, i] - L[:, i, k] * y[:, k]
        y[:, i] = y[:, i] / L[:, i, i]
    for i in range(5, -1, -1):
        for k in range(i + 1, 6):
            y[:, i] = y[:, i] - L[:, k, i] * y[:, k]
        y[:, i] = y[:, i] / L[:, i, i]
    assert np.array_equal(x, y)
