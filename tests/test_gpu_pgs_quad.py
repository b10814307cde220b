"""The contact solver's four-lanes-per-problem kernels where they can go wrong:
batches around a wavefront's sixteen problems, rows around the quads of
columns, a start that is infinite, a zero diagonal, a problem that is not a
number beside others.  Against the sweeps written out in numpy."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from helpers import rel
from test_gpu_pgs import _batch

pytestmark = pytest.mark.gpu


def sweeps(A, b, lo, hi, x, niter):
    with np.errstate(all="ignore"):
        for _ in range(niter):
            for i in range(b.shape[1]):
                o = [j for j in range(b.shape[1]) if j != i]
                y = -(b[:, i] + np.einsum("bj,bj->b", A[:, i, o], x[:, o])) / A[:, i, i]
                x[:, i] = np.where(y < lo[:, i], lo[:, i], np.where(y > hi[:, i], hi[:, i], y))
    return x


def run(A, b, lo, hi, x0, niter, xbar):
    from paper_2109_07719_amd import pgs
    t = [torch.tensor(v, device="cuda") for v in (A, b, lo, hi, x0)]
    ws = pgs.new_workspace(*A.shape[:2], niter, t[0].dtype)
    x = pgs.solve(*t, niter, workspace=ws)
    out = pgs.adjoint(*t[:4], torch.tensor(xbar, device="cuda"), niter, ws)
    return [v.cpu().numpy() for v in (x, *out)]


@pytest.mark.parametrize("n", [1, 3, 4, 5, 8, 9, 12, 13, 16])
@pytest.mark.parametrize("B", [1, 15, 17, 65])
def test_batches_and_rows_around_the_quads(B, n):
    a = _batch(B, n, 7 * n + B, torch.float64)
    xbar = np.random.default_rng(n).normal(size=(B, n))
    print("case", B, n, flush=True)
    got = run(*a, 5, xbar)
    for p in range(B):
        x, sw = O.pgs_solve(*(v[p] for v in a), 5, sweeps=True)
        ref = (x, *O.pgs_adjoint(*(v[p] for v in a[:4]), sw, xbar[p]))
        # round-off of 5 n rows of n terms each
        for g, r in zip(got, ref):
            assert rel(g[p], r, 1e-12) < 1e-13 * 5 * n


@pytest.mark.parametrize("n", [4, 7, 16])
def test_infinite_starts_zero_diagonals_and_a_bad_neighbour(n):
    A, b, lo, hi, x0 = _batch(9, n, 3, torch.float64)
    xbar = np.random.default_rng(1).normal(size=(9, n))
    clean = run(A, b, lo, hi, x0, 4, xbar)
    x0[2, 0] = np.inf          # row 0 does not read it, and replaces it
    A[4, n - 1, n - 1] = 0.0   # the last row goes to a bound
    A[3, 1, 1], hi[3, 1], lo[3, 1] = 0.0, np.inf, -np.inf   # and so does one without bounds
    lo[3, 2:], hi[3, 2:], lo[3, 0], hi[3, 0] = -0.5, 0.5, -0.5, 0.5
    A[6, 1, 2] = np.nan
    got = run(A, b, lo, hi, x0, 4, xbar)
    ref = sweeps(A, b, lo, hi, x0.copy(), 4)
    assert np.isinf(got[0][3, 1]) and np.array_equal(got[0][3], ref[3])
    for p in (2, 4):
        assert rel(got[0][p], ref[p], 1e-12) < 1e-13 * 4 * n
    assert all(np.isfinite(g[2]).all() for g in got[2:])
    for g, r in zip(got, clean):
        keep = [0, 1, 5, 7, 8]
        assert np.array_equal(g[keep], r[keep])
