"""The contact gradient's two-wavefront kernel (small batches) against the
one-wavefront kernel (a batch that fills the chip, of the same systems
repeated): step counts of both parities, a partly filled last wavefront, the
friction gradient, spheres out of contact."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from helpers import rel
from test_gpu_contact_lanes import BETA, DT, G, MU, scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,T", [("star", 2), ("star", 3), ("star", 6), ("free16", 5), ("one", 4)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_two_wavefronts_agree_with_one(kind, T, dtype):
    from paper_2109_07719_amd.contact import ContactBatch
    print("case", kind, T, dtype, flush=True)
    s, q0, qd0, tau, links, centers, radii = scene(kind, 21, T)
    rng = np.random.default_rng(3)
    small, times = 5, 1600   # 8000 systems: two wavefronts each would not be resident
    qd = qd0[:, None] + rng.normal(0, 0.02, (qd0.size, small))
    u = tau[:, :, None] + rng.normal(0, 0.1, (*tau.shape, small))
    q = np.repeat(q0[:, None], small, 1)
    if kind == "star":
        q[1, 3] += 0.5   # off the ground
    gq, gqd = rng.normal(size=q.shape), rng.normal(size=qd.shape)
    got = []
    for n in (1, times):
        f = lambda x: torch.tensor(np.ascontiguousarray(np.tile(x, (1,) * (x.ndim - 1) + (n,))), dtype=dtype, device="cuda")
        cb = ContactBatch([s] * (small * n), links, [centers] * (small * n), [radii] * (small * n), mu=MU, beta=BETA,
                          niter=8, gravity=G, dtype=dtype)
        tr = cb.rollout(f(q), f(qd), f(u), DT)[2]
        got.append([x.cpu().numpy() for x in cb.grad(tr, f(u), DT, f(gq), f(gqd), mu_grad=True)])
    # the same statements, contracted differently at most: FP64 round-off,
    # amplified by the responses of light links, and the FP32 outputs' rounding
    tol = 1e-8 if dtype is torch.float64 else 1e-6
    scale = max(np.abs(a).max() for a in got[0] if a.size)
    for a, b in zip(*got):
        for first in (0, small * (times - 1)):
            b5 = b[..., first:first + small]
            if a.size:
                assert rel(a, b5, 1e-6 * scale) < tol, rel(a, b5, 1e-6 * scale)
