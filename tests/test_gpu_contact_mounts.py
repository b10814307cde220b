"""Contact on fixed bases: where the base stands along the ground changes
nothing."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from contact_cases import grounded_tree

pytestmark = pytest.mark.gpu
G, MU, BETA, DT = (0.0, -9.81, 0.0), 0.7, 0.2, 1e-3


def scene(seed, T, by=(0.0, 0.0)):
    """A tree with random frames, every sphere 1 mm or more under the ground,
    moved along it."""
    s, q0, qd0, tau, links, centers, radii = grounded_tree(seed, T)
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
