"""One step per handle: a rollout's states do not depend on the arithmetic of
the backward pass, and a segment's replay takes the step that the rollout
took, so gradients do not depend on the checkpoint interval."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2109_07719_amd import synth
from test_gpu_frame import turned_chain

pytestmark = pytest.mark.gpu

T = 12
CHAINS = [synth.chain_system(n, 40 + n, T) for n in (3, 7, 20)]


def resized(draws):
    return [(s, q, v, np.resize(u, (T, u.shape[1]))) for s, q, v, u in draws]


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


TURNED = [turned_chain(n, 70 + n) for n in (4, 5, 17)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("K,copies", [(3, 1), (5, 1), (3, 4000)])
def test_replayed_segments_of_turned_chains(dtype, K, copies):
    """Against the gradients from every stored state, for a few batches
    (pipelined) and for many: the same states and statements, compiled apart, so
    each number within a few units of the last place that FP64 round-off can
    move (FP32: of its own)."""
    print("case", dtype, K, copies, flush=True)
    s = setup(resized(TURNED) * copies, dtype)
    got, ref = backward(*s, K), backward(*s, 1, tiling=(1, 1, False))
    assert all(np.array_equal(u, v) for u, v in zip(got[:2], ref[:2]))
    tol = 2.0 ** -22 if dtype is torch.float32 else 1e-13 * 17 ** 3
    for g, r in zip(got[2:], ref[2:]):
        assert (np.abs(g - r) <= tol * np.maximum(np.abs(r), 1e-3 * np.abs(r).max())).all()
