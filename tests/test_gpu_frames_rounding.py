"""Gradients of FP32 handles whose joint frames and ball quaternions are
rounded to FP32, so orthogonal (of unit length) only to 6e-8: as close to the
gradient at the unrounded frames as FP32 outputs can show."""
from dataclasses import replace

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from helpers import rel
from paper_2109_07719_amd import synth

pytestmark = pytest.mark.gpu


def turned_tree(seed, n, ball):
    draw = synth.ball_tree_system if ball else synth.tree_system
    s, q, v, u = draw(seed, 1, nmin=n, nmax=n, random_frames=True)
    rng = np.random.default_rng(seed)
    ax = rng.normal(size=s.axis.shape)
    return replace(s, axis=ax / np.linalg.norm(ax, axis=1, keepdims=True)), q, v, u


@pytest.mark.parametrize("ball", [False, True])
@pytest.mark.parametrize("n,tiling", [(7, None), (23, None), (40, (1, 1, False))])
def test_one_step_gradient_in_fp32(n, tiling, ball):
    """Median relative error of tau_bar over 30 trees below the unit roundoff
    of FP32, 2^-24: inputs and outputs are each off by half of it at most."""
    from paper_2109_07719_amd.sim import Sim
    b = synth.make_batch([turned_tree(300 + k, n, ball) for k in range(30)], 1e-2)
    print("case", n, tiling, ball, flush=True)
    sim = Sim(b.systems, b.gravity, dtype=torch.float32)
    if tiling:
        sim.set_tiling(*tiling)
    r32 = lambda x: np.asarray(x, dtype=np.float32).astype(np.float64)
    rng = np.random.default_rng(3)
    q0, qd0, tau, a, c = map(r32, (b.q0, b.qd0, b.tau, rng.normal(size=sim.nq), rng.normal(size=sim.nv)))
    f = lambda x: torch.tensor(np.ascontiguousarray(x), dtype=torch.float32, device="cuda")
    ws = sim.new_workspace(1, 1)
    sim.forward(f(q0), f(qd0), f(tau), b.dt, K=1, workspace=ws)
    gtau = sim.backward(f(tau), b.dt, 1, ws, f(a), f(c))[2].cpu().numpy()
    oq, ov, ou = b.offsets()
    dt = float(np.float32(b.dt))
    err = []
    for k, s in enumerate(b.systems):
        q, v, u = slice(oq[k], oq[k + 1]), slice(ov[k], ov[k + 1]), slice(ou[k], ou[k + 1])
        g = O.rollout_grad(O.Model(s, b.gravity), q0[q], qd0[v], tau[:, u], dt, a[q], c[v])
        err.append(rel(gtau[:, u], g[2]))
    assert np.median(err) < 2.0 ** -24, np.median(err)
