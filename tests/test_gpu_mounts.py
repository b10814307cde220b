"""Where a system stands changes nothing: a fixed base's dynamics do not
depend on its mounting point, so results far from the origin are those at the
origin.  And the rollout's states do not depend on the checkpoint interval
(store-all, K = 0, is a kernel of its own, which the compiler may contract
otherwise)."""
from dataclasses import replace

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from helpers import rel
from paper_2109_07719_amd import synth

pytestmark = pytest.mark.gpu

T = 6
FAR = np.array([600.0, -300.0, 700.0])
FAMILIES = {
    "trees": [synth.tree_system(80 + k, T, nmin=4, nmax=20, random_frames=True, prismatic=0.2 * k) for k in range(3)],
    "balls": [synth.ball_tree_system(64, T, nmin=9, nmax=20, random_frames=True, prismatic=0.3)],
    "quads": [synth.quadruped_system(96, T)],
    "chains": [synth.chain_system(n, 31, T) for n in (2, 7, 20)],
}


def moved(draws, by):
    """Every root link with a fixed base mounted `by` further off."""
    out = []
    for s, q, v, u in draws:
        r = np.array(s.r_T, dtype=np.float64)
        r[(s.parent < 0) & (s.jtype != synth.FREE)] += by
        out.append((replace(s, r_T=r), q, v, u))
    return out


def sim_of(draws, dtype):
    from paper_2109_07719_amd.sim import Sim
    b = synth.make_batch(draws, 1e-3)
    f = lambda x: torch.tensor(np.ascontiguousarray(x), dtype=dtype, device="cuda")
    return Sim(b.systems, (1.0, -9.0, 2.0), dtype=dtype), f(b.q0), f(b.qd0), f(b.tau), b.dt


def states(draws, dtype, K, ws=True):
    sim, q, v, u, dt = sim_of(draws, dtype)
    w = sim.new_workspace(T, K) if ws else None
    return [x.cpu().numpy() for x in sim.forward(q, v, u, dt, K=K, workspace=w, traj=True)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("name", ["trees", "balls", "quads", "chains"])
def test_forward_does_not_depend_on_the_mount_or_the_interval(name, dtype):
    print("case", name, dtype, flush=True)
    ref = states(FAMILIES[name], dtype, 1, ws=False)
    for draws, K in ((FAMILIES[name], 3), (FAMILIES[name], -2), (moved(FAMILIES[name], FAR), 1)):
        for a, r in zip(states(draws, dtype, K), ref):
            assert np.array_equal(a, r), K


def gradients(draws, dtype, K, tiling=None):
    sim, q, v, u, dt = sim_of(draws, dtype)
    if tiling:
        sim.set_tiling(*tiling)
    rng = np.random.default_rng(5)
    f = lambda *n: torch.tensor(rng.normal(size=n), dtype=dtype, device="cuda")
    a, b, t = f(sim.nq), f(sim.nv), f(T, sim.nq + sim.nv)
    ws = sim.new_workspace(T, K)
    sim.forward(q, v, u, dt, K=K, workspace=ws)
    return [x.cpu().numpy() for x in (*sim.backward(u, dt, K, ws, a, b, t), a, b)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("name", ["trees", "balls", "chains"])
@pytest.mark.parametrize("K,tiling", [(1, None), (1, (1, 1, False)), (3, None), (-2, None)])
def test_gradients_do_not_depend_on_the_mount(name, dtype, K, tiling):
    print("case", name, dtype, K, tiling, flush=True)
    for a, r in zip(gradients(moved(FAMILIES[name], FAR), dtype, K, tiling),
                    gradients(FAMILIES[name], dtype, K, tiling)):
        assert np.array_equal(a, r)


def gantry(seed):
    """Two crossed prismatic joints, the second 1 km out, carrying an arm."""
    s, q, v, u = synth.tree_system(seed, T, nmin=8, nmax=8, random_frames=True)
    parent, jtype, axis = np.arange(8) - 1, np.array(s.jtype), np.array(s.axis)
    jtype[:2] = synth.PRISMATIC
    axis[:2] = np.eye(3)[:2]
    q = np.array(q)
    q[:2] = 700.0, 1000.0
    return replace(s, parent=parent, jtype=jtype, axis=axis), q, v, u


@pytest.mark.parametrize("K", [1, 3])
def test_fp64_gradients_behind_a_long_travel(K):
    """Against the oracle, in FP64 round-off (1e-13 of the link count cubed, as
    for the other adjoint tests)."""
    draws = [gantry(11 + k) for k in range(3)]
    print("case gantry", K, flush=True)
    gq, gqd, gtau, a, b = gradients(draws, torch.float64, K)
    bat = synth.make_batch(draws, 1e-3)
    rng = np.random.default_rng(5)
    t = [rng.normal(size=n) for n in (a.size, b.size, (T, a.size + b.size))][2]
    oq, ov, ou = bat.offsets()
    for k, s in enumerate(bat.systems):
        m = O.Model(s, (1.0, -9.0, 2.0))
        q, v, u = slice(oq[k], oq[k + 1]), slice(ov[k], ov[k + 1]), slice(ou[k], ou[k + 1])
        seed = np.concatenate([t[:, q], t[:, oq[-1] + ov[k]:oq[-1] + ov[k + 1]]], axis=1)
        g = O.rollout_grad(m, bat.q0[q], bat.qd0[v], bat.tau[:, u], bat.dt, a[q], b[v], seed)
        for x, r in zip((gq[q], gqd[v], gtau[:, u]), g):
            assert rel(x, r, 1e-12) < 1e-13 * s.n ** 3, (k, rel(x, r, 1e-12))
