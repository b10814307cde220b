"""The contact solver on both sides of the batch from which problems of up to
four rows take a lane each (16 problems per SIMD), against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from helpers import rel
from test_gpu_pgs import _batch
from test_gpu_pgs_quad import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("more", [0, 1, 63])
def test_around_a_lane_per_problem(n, more, dtype):
    B = 16 * 4 * torch.cuda.get_device_properties(0).multi_processor_count + more
    few = 97                       # that many different problems, over and over
    f = np.float64 if dtype is torch.float64 else np.float32
    base = [v.astype(f) for v in _batch(few, n, 5 * n + more, dtype)]
    a = [np.ascontiguousarray(v[np.arange(B) % few]) for v in base]
    xbar = np.random.default_rng(n).normal(size=(B, n)).astype(f)
    print("case", B, n, dtype, flush=True)
    got = run(*a, 5, xbar)
    wide = [v.astype(np.float64) for v in a]
    # round-off of 5 n rows of n terms each, amplified by the problems' own
    # condition in FP32 as in FP64
    tol = 1e-13 * 5 * n * (1 if dtype is torch.float64 else 2.0 ** 29)
    for p in [*range(8), *range(B - 70, B)]:
        x, sw = O.pgs_solve(*(v[p] for v in wide), 5, sweeps=True)
        ref = (x, *O.pgs_adjoint(*(v[p] for v in wide[:4]), sw, xbar[p].astype(np.float64)))
        for g, r in zip(got, ref):
            assert rel(g[p], r, 1e-12 if dtype is torch.float64 else 1e-6) < tol
