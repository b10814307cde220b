"""Serial chains with parallel axes (the planar kernels) where they can go
wrong: one link, the lane counts around the switch from level steps to lane
scans (16 and 17 levels), the longest chain, several lengths in one wavefront;
horizons around the pipeline's phases; every checkpointing scheme; a diverged
neighbour.  Against the FP64 oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from helpers import rel
from paper_2109_07719_amd import synth

pytestmark = pytest.mark.gpu


def batch(sizes, T, seed):
    draws = [synth.chain_system(n, seed + k, T) for k, n in enumerate(sizes)]
    rng = np.random.default_rng(seed)
    for k, (s, *_) in enumerate(draws):   # offsets and masses off the x axis
        s.r_T[1:] += rng.normal(0, 0.1, (s.n - 1, 3))
        s.com[:] += rng.normal(0, 0.1, (s.n, 3))
        s.Ic[:, 3:] = rng.normal(0, 0.002, (s.n, 3))
    return synth.make_batch(draws, 1e-3)


def run(b, K, dtype=torch.float64, tiling=None):
    from paper_2109_07719_amd.sim import Sim
    sim = Sim(b.systems, (1.0, -9.0, 2.0), dtype=dtype)
    assert sim.info["chain"] and sim.info["frames_identity"]
    if tiling:
        sim.set_tiling(*tiling)
    f = lambda x: torch.tensor(np.ascontiguousarray(x), dtype=dtype, device="cuda")
    q0, qd0, tau = f(b.q0), f(b.qd0), f(b.tau)
    rng = np.random.default_rng(5)
    gq, gqd = f(rng.normal(size=sim.nq)), f(rng.normal(size=sim.nv))
    gt = f(rng.normal(size=(b.T, sim.nq + sim.nv)))
    ws = sim.new_workspace(b.T, K)
    qT, qdT, _ = sim.forward(q0, qd0, tau, b.dt, K=K, workspace=ws)
    out = sim.backward(tau, b.dt, K, ws, gq, gqd, gt)
    return [x.cpu().numpy() for x in (qT, qdT, *out)], [x.cpu().numpy() for x in (gq, gqd, gt)], sim.aba(q0, qd0, tau[0].contiguous())


@pytest.mark.parametrize("sizes", [(1, 1, 2), (7, 1, 16, 17), (64, 3), (9, 50, 5)])
@pytest.mark.parametrize("T,K,tiling", [(1, 1, None), (2, 1, None), (5, 1, (1, 2, True)), (6, 1, (2, 1, False)),
                                        (7, 3, None), (7, -2, None)])
def test_planar_chains_fp64(sizes, T, K, tiling):
    print("case", sizes, T, K, tiling, flush=True)
    b = batch(sizes, T, 40)
    got, (gq, gqd, gt), qdd = run(b, K, tiling=tiling)
    oq, ov, ou = b.offsets()
    nq = oq[-1]
    for k, s in enumerate(b.systems):
        m = O.Model(s, (1.0, -9.0, 2.0))
        q, u = slice(oq[k], oq[k + 1]), slice(ou[k], ou[k + 1])
        seed = np.concatenate([gt[:, q], gt[:, nq + oq[k]:nq + oq[k + 1]]], axis=1)
        g = O.rollout_grad(m, b.q0[q], b.qd0[q], b.tau[:, u], b.dt, gq[q], gqd[q], seed)
        ref = [g[3], g[4], g[0], g[1], g[2]]
        mine = [got[0][q], got[1][q], got[2][q], got[3][q], got[4][:, u]]
        # FP64 round-off of two evaluation orders; a chain's inertia matrix
        # has a condition of about n^4
        tol = 1e-13 * max(s.n, 4) ** 3
        for a, r in zip(mine, ref):
            assert rel(a, r, 1e-12) < tol, (s.n, rel(a, r, 1e-12))
        a = qdd[q].cpu().numpy()
        assert rel(a, O.fd(m, b.q0[q], b.qd0[q], b.tau[0, u]), 1e-12) < tol


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_a_diverged_chain_leaves_its_neighbours_alone(dtype):
    b = batch((7, 7, 7, 20, 7), 4, 60)
    clean, *_ = run(b, 1, dtype)
    b.qd0[7:14] = 1e30
    for tiling in (None, (4, 1, False)):
        got, *_ = run(b, 1, dtype, tiling)
        assert not np.isfinite(got[0][7:14]).all()
        keep = np.r_[0:7, 14:b.q0.size]
        ref = clean if tiling is None else run(batch((7, 7, 7, 20, 7), 4, 60), 1, dtype, tiling)[0]
        for a, r in zip(got, ref):
            assert np.array_equal(a[..., keep], r[..., keep])
