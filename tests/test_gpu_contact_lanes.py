"""The contact kernels at the edges of their lane layout (16 lanes per system,
four systems per wavefront, lane = link or contact row), against the FP64
oracle: one link, the largest chains and free-root trees, spheres on the free
root and two on one link, no and the most recorded sweeps, batches that leave
a wavefront partly filled, no steps."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from helpers import rel
from paper_2109_07719_amd import synth

pytestmark = pytest.mark.gpu
G, MU, BETA, DT = (0.0, -9.81, 0.0), 0.7, 0.2, 1e-3


def scene(kind, seed, T):
    rng = np.random.default_rng(seed)
    if kind == "one":
        n, links, free = 1, [0], False
    elif kind == "chain16":
        n, links, free = 16, [15, 7, 7, 0], False
    elif kind == "free16":
        n, links, free = 16, [0, 15, 9, 9], True
    elif kind == "free1":
        n, links, free = 1, [0, 0], True
    else:  # a star: every link on the root
        n, links, free = 9, [1, 4, 4, 8], True
    parent = np.array([-1] + [0 if kind == "star" else i if kind == "chain16" else int(rng.integers(max(0, i - 2), i + 1))
                              for i in range(n - 1)], np.int32)
    jt = np.where(np.random.default_rng(7).uniform(size=n) < 0.3, synth.PRISMATIC, synth.REVOLUTE).astype(np.int32)
    if free:
        jt[0] = synth.FREE
    unit = lambda v: v / np.linalg.norm(v, axis=-1, keepdims=True)
    Ic = np.zeros((n, 6))
    Ic[:, :3] = rng.uniform(0.01, 0.1, (n, 3))
    s = synth.System(parent=parent, jtype=jt, E_T=np.tile(np.eye(3), (n, 1, 1)), r_T=0.2 * unit(rng.normal(size=(n, 3))),
                     axis=unit(rng.normal(size=(n, 3))), mass=rng.uniform(0.5, 2, n), com=rng.uniform(-0.1, 0.1, (n, 3)),
                     Ic=Ic)
    q0, qd0 = rng.normal(0, 0.1, s.nq), rng.normal(0, 0.1, s.nv)
    if free:
        q0[3:7] = unit(np.r_[0.2 * rng.normal(size=3), 1.0])
    # radii that sink every sphere a little: the height of its centre plus 1 mm
    m = O.Model(s, G)
    centers, radii = rng.normal(0, 0.1, (len(links), 3)), np.full(len(links), 1e6)
    _, phi, _, _ = O.contact_assembly(m, O.Contacts(links, centers, radii), q0)
    if free:
        q0[1] -= (phi + 1e6).min() - 0.05
        phi = phi - ((phi + 1e6).min() - 0.05)
    else:
        s.r_T[0, 1] -= (phi + 1e6).min() - 0.05
        phi = phi - ((phi + 1e6).min() - 0.05)
    radii = phi + 1e6 + rng.uniform(5e-4, 2e-3, len(links))
    return s, q0, qd0, rng.normal(0, 0.3, (T, s.nu)), np.array(links, np.int32), centers, radii


@pytest.mark.parametrize("kind,B,T,niter", [("one", 1, 3, 5), ("chain16", 5, 4, 20), ("free16", 3, 4, 64),
                                            ("free1", 2, 4, 10), ("star", 6, 3, 30), ("star", 4, 2, 0),
                                            ("free16", 2, 0, 8)])
def test_lane_layout_edges_fp64(kind, B, T, niter):
    from paper_2109_07719_amd.contact import ContactBatch
    print("case", kind, B, T, niter, flush=True)
    # one topology: the same structure stream, other numbers per system
    base = scene(kind, 11, T)
    draws = []
    for i in range(B):
        r = np.random.default_rng(100 + i)
        s, q0, qd0, tau, links, centers, radii = scene(kind, 11, T)
        s.mass = s.mass * r.uniform(0.8, 1.2, s.n)
        draws.append((s, q0, qd0 + r.normal(0, 0.02, qd0.shape), tau + r.normal(0, 0.1, tau.shape), links, centers, radii))
    cb = ContactBatch([d[0] for d in draws], base[4], [d[5] for d in draws], [d[6] for d in draws], mu=MU, beta=BETA,
                      niter=niter, gravity=G, dtype=torch.float64)
    f = lambda k: torch.tensor(np.ascontiguousarray(np.stack([d[k] for d in draws], -1)), device="cuda")
    q0, qd0, tau = f(1), f(2), f(3)
    qT, qdT, tr, nc = cb.rollout(q0, qd0, tau, DT, counts=True)
    rng = np.random.default_rng(3)
    gq, gqd = (torch.tensor(rng.normal(size=x.shape), device="cuda") for x in (qT, qdT))
    g = [x.cpu().numpy() for x in cb.grad(tr, tau, DT, gq, gqd, mu_grad=True)]
    # the bars of the FP64 tests of larger batches: round-off of two
    # evaluation orders, amplified by the responses of light links
    for i, d in enumerate(draws):
        m, C = O.Model(d[0], G), O.Contacts(d[4], d[5], d[6], mu=MU, beta=BETA, niter=niter)
        rq, rqd, rnc = O.rollout_contact(m, C, d[1], d[2], d[3], DT)
        assert np.array_equal(nc[:, i].cpu().numpy(), rnc)
        assert T == 0 or rnc[0] == len(d[4])
        assert rel(qT[:, i].cpu().numpy(), rq, 1e-12) < 1e-10 and rel(qdT[:, i].cpu().numpy(), rqd, 1e-12) < 1e-10
        ref = O.rollout_contact_grad(m, C, d[1], d[2], d[3], DT, gq[:, i].cpu().numpy(), gqd[:, i].cpu().numpy(),
                                     mu_grad=True)
        ref = ref[:3] + (np.array([ref[3]]),)
        got = [g[0][:, i], g[1][:, i], g[2][:, :, i], g[3][i:i + 1]]
        if d[0].jtype[0] == synth.FREE:
            # off the unit sphere two readings of R differ: compare along it
            qt = d[1][3:7] / np.linalg.norm(d[1][3:7])
            for v in (got, ref):
                v[0][3:7] -= (v[0][3:7] @ qt) * qt
        scale = max([np.abs(r).max() for r in ref if r.size])
        for a, b in zip(got, ref):
            assert a.size == 0 or rel(a, b, 1e-6 * scale) < 1e-8
