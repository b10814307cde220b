"""Contact on fixed bases: where the base stands along the ground changes
nothing, and FP32 batches, whose joint frames are orthogonal only to 6e-8,
give gradients as close to those at the unrounded frames as FP32 outputs can
show."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from contact_cases import grounded_tree
from helpers import rel
from paper_2109_07719_amd import synth

pytestmark = pytest.mark.gpu
G, MU, BETA, DT = (0.0, -9.81, 0.0), 0.7, 0.2, 1e-3


def scene(seed, T, by=(0.0, 0.0), n=None):
    """A tree with random frames, every sphere 1 mm or more under the ground,
    moved along it."""
    s, q0, qd0, tau, links, centers, radii = grounded_tree(seed, T)
    if n:
        s, q0, qd0, tau = synth.tree_system(seed, T, nmin=n, nmax=n, random_frames=True, max_depth=n)
        links = np.linspace(n // 2, n - 1, 4).astype(np.int32)
    _, phi, _, _ = O.contact_assembly(O.Model(s, G), O.Contacts(links, centers, np.full(4, 1e6)), q0)
    s.r_T[0] -= (0.0, (phi + 1e6 - radii).max() + 1e-3, 0.0)
    s.r_T[0] += (by[0], 0.0, by[1])
    return s, q0, qd0, tau, links, centers, radii


def run(d, dtype):
    from paper_2109_07719_amd.contact import ContactBatch
    cb = ContactBatch([d[0]], d[4], [d[5]], [d[6]], mu=MU, beta=BETA, niter=20, gravity=G, dtype=dtype)
    f = lambda x: torch.tensor(np.ascontiguousarray(np.asarray(x)[..., None]), dtype=dtype, device="cuda")
    rng = np.random.default_rng(3)
    a, b = f(rng.normal(size=d[0].nq)), f(rng.normal(size=d[0].nv))
    qT, qdT, tr, nc = cb.rollout(f(d[1]), f(d[2]), f(d[3]), DT, counts=True)
    g = cb.grad(tr, f(d[3]), DT, a, b, mu_grad=True)
    assert int(nc[0, 0]) == 4
    return [x.cpu().numpy()[..., 0] for x in (qT, qdT, tr, *g, a, b)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_results_do_not_depend_on_the_place_along_the_ground(dtype):
    T = 4
    for seed in range(5):
        print("case", dtype, seed, flush=True)
        for a, r in zip(run(scene(seed, T, (600.0, -700.0)), dtype), run(scene(seed, T), dtype)):
            assert np.array_equal(a, r)


@pytest.mark.parametrize("n", [8, 16])
def test_one_step_gradient_in_fp32(n):
    """Median relative error of tau_bar over 30 trees below the unit roundoff
    of FP32, 2^-24: inputs and outputs are each off by half of it at most."""
    r32 = lambda x: np.asarray(x, dtype=np.float32).astype(np.float64)
    err = []
    for seed in range(30):
        d = list(scene(seed, 1, n=n))
        d[1:4] = map(r32, d[1:4])
        print("case", n, seed, flush=True)
        out = run(d, torch.float32)
        m, C = O.Model(d[0], G), O.Contacts(d[4], d[5], d[6], mu=MU, beta=BETA, niter=20)
        g = O.rollout_contact_grad(m, C, d[1], d[2], d[3], float(np.float32(DT)), *out[-2:])
        err.append(rel(out[5], g[2]))
    assert np.median(err) < 2.0 ** -24, np.median(err)
