"""One step per handle: a rollout's states do not depend on the arithmetic of
the backward pass."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2109_07719_amd import synth

pytestmark = pytest.mark.gpu

T = 12
CHAINS = [synth.chain_system(n, 40 + n, T) for n in (3, 7, 20)]


def setup(draws, dtype):
    from paper_2109_07719_amd.sim import Sim
    b = synth.make_batch(draws, 1e-3)
    sim = Sim(b.systems, (1.0, -9.0, 2.0), dtype=dtype)
    f = lambda x: torch.tensor(np.ascontiguousarray(x), dtype=dtype, device="cuda")
    rng = np.random.default_rng(5)
    return sim, (f(b.q0), f(b.qd0), f(b.tau)), b.dt, (f(rng.normal(size=sim.nq)), f(rng.normal(size=sim.nv)))


def backward(sim, x, dt, seeds, K, before=None, after=None, tiling=None):
    """Forward with one adjoint dtype set, backward with another."""
    if tiling:
        sim.set_tiling(*tiling)
    ws = sim.new_workspace(T, K)
    if before:
        sim.set_adjoint_dtype(before)
    end = sim.forward(*x, dt, K=K, workspace=ws)[:2]
    if after:
        sim.set_adjoint_dtype(after)
    return [v.cpu().numpy() for v in (*end, *sim.backward(x[2], dt, K, ws, *seeds))]


@pytest.mark.parametrize("K", [1, 0, 3, -2])
def test_the_adjoint_dtype_leaves_the_forward_alone(K):
    print("case", K, flush=True)
    s = setup(CHAINS, torch.float32)
    f32, f64 = torch.float32, torch.float64
    a, b = backward(*s, K, f64, f64), backward(*s, K, f32, f32)
    assert all(np.array_equal(u, v) for u, v in zip(a[:2], b[:2]))
    # a change in between reverses the rollout that ran: the gradients of the
    # handle that had the last dtype all along
    for before, after, ref in ((f32, f64, a), (f64, f32, b)):
        got = backward(*s, K, before, after)
        assert all(np.array_equal(u, v) for u, v in zip(got, ref))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_end_states_of_chains_do_not_depend_on_the_interval(dtype):
    s = setup(CHAINS, dtype)
    ref = backward(*s, 1)[:2]
    for K in (0, 3, -2):
        assert all(np.array_equal(u, v) for u, v in zip(backward(*s, K)[:2], ref)), K
