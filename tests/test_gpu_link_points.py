"""Link points on the GPU kernels against the torch expressions of the same
module: every joint type, path lengths around the scan's rounds (1, 2, 3, 64
links, and 65, which the kernels do not take), and the calls that must keep
running the torch expressions (second derivatives, forward mode, vmap)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2109_07719_amd import synth
from paper_2109_07719_amd.fk import LinkPoints, _paths

G = torch.device("cuda")


def system(n, seed, types=(0, 2, 3), free=False):
    rng = np.random.default_rng(seed)
    unit = lambda v: v / np.linalg.norm(v, axis=-1, keepdims=True)
    jt = rng.choice(types, n).astype(np.int32)
    if free:
        jt[0] = synth.FREE
    ET = np.stack([np.linalg.qr(rng.normal(size=(3, 3)))[0] for _ in range(n)])
    parent = np.array([-1] + [i if rng.random() < 0.9 else int(rng.integers(0, i + 1)) for i in range(n - 1)], np.int32)
    s = synth.System(parent=parent, jtype=jt, E_T=ET, r_T=0.3 * rng.normal(size=(n, 3)), axis=unit(rng.normal(size=(n, 3))),
                     mass=np.ones(n), com=np.zeros((n, 3)), Ic=np.tile([1, 1, 1, 0, 0, 0.0], (n, 1)))
    return s


def test_paths():
    par, jt = np.array([-1, 0, 1, 1, -1, 4]), np.zeros(6, int)
    assert _paths(np.array([3, 5, 0]), par, jt).tolist() == [[0, 1, 3], [4, 5, -1], [0, -1, -1]]
    assert _paths(np.array([-1]), par, jt).tolist() == [[4, 5]]
    assert _paths(np.array([6]), par, jt) is None and _paths(np.array([3]), par, jt, most=2) is None
    jt[1] = 1
    assert _paths(np.array([3]), par, jt).tolist() == [[1, 3]]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("sizes", [(1,), (2, 1, 3), (3, 7, 13, 5, 8), (64, 2), (65, 4)])
def test_kernel_equals_torch(sizes, dtype):
    sys_ = [system(n, 10 + k, free=k % 2 == 1) for k, n in enumerate(sizes)]
    if max(sizes) >= 64:   # a chain: the path is the whole system
        sys_[0].parent = np.arange(-1, sizes[0] - 1, dtype=np.int32)
    rng = np.random.default_rng(1)
    fk = LinkPoints(sys_, [s.n - 1 for s in sys_], rng.normal(size=(len(sizes), 3)), dtype=dtype)
    nq = sum(s.nq for s in sys_)
    q = torch.tensor(rng.normal(size=nq), dtype=dtype, device=G, requires_grad=True)
    g = torch.tensor(rng.normal(size=(len(sizes), 3)), dtype=dtype, device=G)
    assert fk._native(q) == (max(sizes) <= 64)
    x, ref = fk(q), fk._positions(q)
    (gq,), (gr,) = torch.autograd.grad(x, q, g), torch.autograd.grad(ref, q, g)
    # unnormalised quaternions scale a path by |quat|^2 a joint: errors are
    # relative to the largest entry; a path of n maps rounds n times
    eps = torch.finfo(dtype).eps * 40 * max(sizes)
    assert (x - ref).abs().max() <= eps * ref.abs().max()
    assert (gq - gr).abs().max() <= eps * gr.abs().max()


@pytest.mark.gpu
def test_other_calls_keep_the_torch_expressions():
    s = system(5, 3, types=(0,))
    fk = LinkPoints([s, s], [4, 2], [[0.5, 0, 0], [0, 0.1, 0]], dtype=torch.float64)
    q = torch.randn(10, dtype=torch.float64, device=G, requires_grad=True)
    assert torch.autograd.gradgradcheck(lambda v: fk(v), (q,))
    _, t = torch.func.jvp(fk, (q.detach(),), (torch.ones_like(q),))
    eps = 1e-6
    fd = (fk(q.detach() + eps) - fk(q.detach() - eps)) / (2 * eps)
    assert (t - fd).abs().max() < 1e-8
    both = torch.func.vmap(fk)(torch.stack([q.detach(), 2 * q.detach()]))
    assert torch.allclose(both[1], fk(2 * q.detach()))
    assert fk(q.detach()[::1].repeat_interleave(2)[::2]).shape == (2, 3)
