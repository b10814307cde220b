"""Gradients where the inputs are not quite what they stand for: ball and root
quaternions off the unit sphere (the step scales the joint's transform by
|quat|^2) and joint frames that are rotations only to a few digits.  Both are
part of the step, so its gradient is that of what the step does."""
from dataclasses import replace

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from helpers import emu_rollout_grad, rel
from paper_2109_07719_amd import synth

pytestmark = pytest.mark.gpu

T = 3


def scaled_quats(s, q, scale):
    q, i = np.array(q), 0
    for j in s.jtype:
        if j in (synth.FREE, synth.SPHERICAL):
            o = i + (3 if j == synth.FREE else 0)
            q[o:o + 4] *= scale
            i = o + 4
        else:
            i += 1
    return q


def check(draws, K, tiling, tol, dtype=torch.float64):
    """Against the sequential reversed statements in FP64."""
    from paper_2109_07719_amd.sim import Sim
    b = synth.make_batch(draws, 1e-2)
    sim = Sim(b.systems, b.gravity, dtype=dtype)
    if tiling:
        sim.set_tiling(*tiling)
    rng = np.random.default_rng(3)
    n = lambda *k: rng.normal(size=k).astype(np.float32).astype(np.float64)
    a, c = n(sim.nq), n(sim.nv)
    f = lambda x: torch.tensor(np.ascontiguousarray(x), dtype=dtype, device="cuda")
    ws = sim.new_workspace(T, K)
    sim.forward(f(b.q0), f(b.qd0), f(b.tau), b.dt, K=K, workspace=ws)
    got = [x.cpu().numpy() for x in sim.backward(f(b.tau), b.dt, K, ws, f(a), f(c))]
    oq, ov, ou = b.offsets()
    for k, s in enumerate(b.systems):
        q, v, u = slice(oq[k], oq[k + 1]), slice(ov[k], ov[k + 1]), slice(ou[k], ou[k + 1])
        g = emu_rollout_grad(s, b.q0[q], b.qd0[v], b.tau[:, u], b.dt, a[q], c[v], gravity=b.gravity)
        for x, r in zip((got[0][q], got[1][v], got[2][:, u]), g):
            if r.size:
                assert rel(x, r, 1e-12) < tol * max(s.n, 4) ** 3, (k, s.n, rel(x, r, 1e-12))


@pytest.mark.parametrize("scale", [1.0 + 1e-4, 1.05])
@pytest.mark.parametrize("K,tiling", [(1, None), (1, (1, 1, False)), (2, None), (-1, None)])
def test_quaternions_off_the_unit_sphere(K, tiling, scale):
    print("case", K, tiling, scale, flush=True)
    draws = [synth.ball_tree_system(64, T, nmin=9, nmax=20, random_frames=True, prismatic=0.3),
             synth.ball_quadruped_system(63, T), synth.quadruped_system(62, T)]
    check([(s, scaled_quats(s, q, scale), v, u) for s, q, v, u in draws], K, tiling, 1e-13)


@pytest.mark.parametrize("K,tiling", [(1, None), (1, (1, 1, False)), (2, None), (-1, None)])
@pytest.mark.parametrize("digits", [3, 7])
def test_frames_of_few_digits(K, tiling, digits):
    print("case", K, tiling, digits, flush=True)
    draws = [synth.tree_system(80 + k, T, nmin=6, nmax=20, random_frames=True, prismatic=0.2 * k) for k in range(2)]
    check([(replace(s, E_T=np.round(s.E_T, digits)), q, v, u) for s, q, v, u in draws], K, tiling, 1e-13)
