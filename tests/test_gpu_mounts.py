"""Where a system stands changes nothing: a fixed base's dynamics do not
depend on its mounting point, so results far from the origin are those at the
origin.  And the rollout's states do not depend on the checkpoint interval
(store-all, K = 0, is a kernel of its own, which the compiler may contract
otherwise)."""
from dataclasses import replace

import numpy as np
import pytest

torch = pytest.importorskip("torch")

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
@pytest.mark.parametrize("name", ["trees", "balls", "quads"])
def test_forward_does_not_depend_on_the_mount_or_the_interval(name, dtype):
    print("case", name, dtype, flush=True)
    ref = states(FAMILIES[name], dtype, 1, ws=False)
    for draws, K in ((FAMILIES[name], 3), (FAMILIES[name], -2), (moved(FAMILIES[name], FAR), 1)):
        for a, r in zip(states(draws, dtype, K), ref):
            assert np.array_equal(a, r), K
