"""Calls of link points that a user makes beyond one gradient: Jacobians with
batched cotangents, a q changed in place after the call, points that share
joints, a module stored by an earlier version."""
import copy

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2109_07719_amd import synth
from paper_2109_07719_amd.fk import LinkPoints

pytestmark = pytest.mark.gpu
G = torch.device("cuda")


def chains(k, n=5):
    return [synth.chain_system(n, 20 + i, 1)[0] for i in range(k)]


def points(k):
    return np.random.default_rng(1).normal(size=(k, 3))


def jacobian(fk, q):
    """Row by row, by the torch expressions."""
    v = q.detach().clone().requires_grad_()
    x = fk._positions(v).reshape(-1)
    return torch.stack([torch.autograd.grad(x[i], v, retain_graph=True)[0] for i in range(x.numel())])


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_batched_cotangents(dtype):
    fk = LinkPoints(chains(2), [4, 2], points(2), dtype=dtype)
    q = torch.randn(10, dtype=dtype, device=G, requires_grad=True)
    assert fk._native(q)
    ref = jacobian(fk, q)
    eye = torch.eye(6, dtype=dtype, device=G).reshape(6, 2, 3)
    tol = dict(rtol=0, atol=40 * 5 * torch.finfo(dtype).eps * float(ref.abs().max()))
    got, = torch.autograd.grad(fk(q), q, eye, is_grads_batched=True)
    assert torch.allclose(got, ref, **tol)
    J = torch.autograd.functional.jacobian(fk, q, vectorize=True)
    assert torch.allclose(J.reshape(6, 10), ref, **tol)
    assert torch.allclose(torch.autograd.functional.jacobian(fk, q).reshape(6, 10), ref, **tol)
    assert torch.allclose(torch.func.jacrev(fk)(q.detach()).reshape(6, 10), ref, **tol)
    assert torch.allclose(torch.func.jacfwd(fk)(q.detach()).reshape(6, 10), ref, **tol)


def test_q_may_change_in_place_after_the_call():
    fk = LinkPoints(chains(2), [4, 2], points(2), dtype=torch.float64)
    q = torch.randn(10, dtype=torch.float64, device=G)
    g = torch.randn(2, 3, dtype=torch.float64, device=G)
    v = q.clone().requires_grad_()
    ref, = torch.autograd.grad(fk._positions(v), v, g)
    leaf = q.clone().requires_grad_()
    x = fk(leaf)
    with torch.no_grad():
        leaf += 1.0
    x.backward(g)
    assert torch.allclose(leaf.grad, ref, rtol=0, atol=1e-13)


@pytest.mark.parametrize("links", [[4, -1], [9, 2], [-10, 0]])
def test_points_that_share_joints_add_up(links):
    """Indices that reach into the neighbouring system, as a negative one does."""
    fk = LinkPoints(chains(2), links, points(2), dtype=torch.float64)
    q = torch.randn(10, dtype=torch.float64, device=G, requires_grad=True)
    g = torch.randn(2, 3, dtype=torch.float64, device=G)
    x, ref = fk(q), fk._positions(q)
    assert torch.allclose(x, ref, rtol=0, atol=1e-13)
    (gq,), (gr,) = torch.autograd.grad(x, q, g), torch.autograd.grad(ref, q, g)
    assert torch.allclose(gq, gr, rtol=0, atol=1e-13)


def test_a_module_without_paths():
    fk = copy.deepcopy(LinkPoints(chains(2), [4, 2], points(2), dtype=torch.float64))
    q = torch.randn(10, dtype=torch.float64, device=G)
    x = fk(q)
    for k in ("_path", "_jtype", "_nq"):   # as stored before the kernels
        del fk.__dict__[k]
    assert torch.allclose(fk(q), x, rtol=0, atol=1e-13)
