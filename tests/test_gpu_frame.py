"""The base-frame FP64 adjoint (trees, free roots, prismatic and ball joints,
limits, chains of any axes) where it can go wrong: one link, a free root
alone, ball joints at a root and at a leaf, the depths around the doubling
rounds' powers of two up to the longest chain, several children and systems in
one wavefront, every checkpointing scheme, a diverged neighbour.  Against the
FP64 oracle."""
from dataclasses import replace

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
from helpers import rel
from paper_2109_07719_amd import synth

pytestmark = pytest.mark.gpu

T = 5


def turned_chain(n, seed):
    s, q, v, u = synth.chain_system(n, seed, T)
    rng = np.random.default_rng(seed)
    E = np.linalg.qr(rng.normal(size=(n, 3, 3)))[0]
    E *= np.sign(np.linalg.det(E))[:, None, None]
    return replace(s, E_T=E.reshape(s.E_T.shape)), q, v, u


def lone_root(seed):
    s, q, v, u = synth.quadruped_system(seed, T)
    cut = {k: getattr(s, k)[:1] for k in ("parent", "jtype", "E_T", "r_T", "axis", "mass", "com", "Ic")}
    return replace(s, **cut), q[:7], v[:6], u[:, :0]


def balls(n, links, seed):
    return synth.with_spherical_joints(*turned_chain(n, seed), links, seed)


DRAWS = {
    "turned_1_2_3": [turned_chain(n, 70 + n) for n in (1, 2, 3)],
    "turned_4_5_17": [turned_chain(n, 70 + n) for n in (4, 5, 17)],
    "turned_64": [turned_chain(64, 7)],
    "prismatic_33": [synth.prismatic_chain_system(33, 8, T)],
    "trees": [synth.tree_system(80 + k, T, nmin=4, nmax=n, max_depth=d, random_frames=k % 2 == 0, prismatic=0.3 * k)
              for k, (n, d) in enumerate(((4, 2), (8, 3), (30, 6)))],
    "limits": [synth.with_joint_limits(synth.tree_system(90, T, nmin=6, nmax=20), 91),
               synth.with_joint_limits(synth.quadruped_system(92, T), 93)],
    "roots": [lone_root(95), synth.quadruped_system(96, T), turned_chain(3, 97), synth.telescoping_quadruped_system(98, T)],
    "balls": [balls(1, (0,), 60), balls(4, (0, 3), 61), balls(6, range(6), 62), synth.ball_quadruped_system(63, T),
              synth.ball_tree_system(64, T, nmin=9, nmax=20, random_frames=True, prismatic=0.3), lone_root(65)],
}


def run(b, K, dtype=torch.float64, tiling=None):
    from paper_2109_07719_amd.sim import Sim
    sim = Sim(b.systems, (1.0, -9.0, 2.0), dtype=dtype)
    if tiling:
        sim.set_tiling(*tiling)
    f = lambda x: torch.tensor(np.ascontiguousarray(x), dtype=dtype, device="cuda")
    tau = f(b.tau)
    rng = np.random.default_rng(5)
    gq, gqd = f(rng.normal(size=sim.nq)), f(rng.normal(size=sim.nv))
    gt = f(rng.normal(size=(b.T, sim.nq + sim.nv)))
    ws = sim.new_workspace(b.T, K)
    sim.forward(f(b.q0), f(b.qd0), tau, b.dt, K=K, workspace=ws)
    out = sim.backward(tau, b.dt, K, ws, gq, gqd, gt)
    return [x.cpu().numpy() for x in out], [x.cpu().numpy() for x in (gq, gqd, gt)]


@pytest.mark.parametrize("name", list(DRAWS))
@pytest.mark.parametrize("K,tiling", [(1, None), (1, (1, 1, False)), (3, None), (5, None), (-2, None)])
def test_base_frame_adjoint_fp64(name, K, tiling):
    print("case", name, K, tiling, flush=True)
    b = synth.make_batch(DRAWS[name], 1e-3)
    got, (gq, gqd, gt) = run(b, K, tiling=tiling)
    oq, ov, ou = b.offsets()
    nq = oq[-1]
    for k, s in enumerate(b.systems):
        m = O.Model(s, (1.0, -9.0, 2.0))
        q, v, u = slice(oq[k], oq[k + 1]), slice(ov[k], ov[k + 1]), slice(ou[k], ou[k + 1])
        seed = np.concatenate([gt[:, q], gt[:, nq + ov[k]:nq + ov[k + 1]]], axis=1)
        # a ball joint's seed along the unit sphere, as the library reads it
        g = O.rollout_grad(m, b.q0[q], b.qd0[v], b.tau[:, u], b.dt, gq[q], gqd[v], seed)
        # FP64 round-off of two evaluation orders; a chain's inertia matrix
        # has a condition of about n^4
        tol = 1e-13 * max(s.n, 4) ** 3
        for a, r in zip((got[0][q], got[1][v], got[2][:, u]), (O.ball_tangent(s, b.q0[q], g[0]), g[1], g[2])):
            if r.size:
                assert rel(a, r, 1e-12) < tol, (k, s.n, rel(a, r, 1e-12))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("name,bad", [("trees", 1), ("roots", 1), ("balls", 3)])
def test_a_diverged_system_leaves_its_neighbours_alone(dtype, name, bad):
    b = synth.make_batch(DRAWS[name], 1e-3)
    clean, _ = run(b, 1, dtype)
    ov = b.offsets()[1]
    b.qd0[ov[bad]:ov[bad + 1]] = 1e30
    got, _ = run(b, 1, dtype)
    for a, r, o in zip(got, clean, b.offsets()):
        keep = np.r_[0:o[bad], o[bad + 1]:o[-1]]
        assert np.array_equal(a[..., keep], r[..., keep])
        assert not np.isfinite(a[..., o[bad]:o[bad + 1]]).all()


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("name", ["turned_4_5_17", "limits", "roots", "balls"])
@pytest.mark.parametrize("T,K", [(1, 1), (2, 1), (9, 1), (9, 4), (12, 4), (3, 4), (9, 2), (9, 40)])
def test_pipelined_wavefronts_agree_with_one(dtype, name, T, K):
    """The pipelined kernels (one batch per workgroup) at horizons around their
    phases and segments, with more systems than one wavefront holds, against
    the one-wavefront kernel at K = 1: the same arithmetic, so the same
    gradients up to how the compiler contracts it, in FP64 round-off (1e-13 of
    the largest link count cubed, as above)."""
    draws = [(s, q, v, np.resize(u, (T, u.shape[1]))) for s, q, v, u in DRAWS[name]] * 5
    b = synth.make_batch(draws, 1e-3)
    print("case", dtype, name, T, K, flush=True)
    got, _ = run(b, K, dtype)
    ref, _ = run(b, 1, dtype, (1, 1, False))
    tol = 1e-13 * 17 ** 3 if dtype is torch.float64 else 1e-6
    for a, r in zip(got, ref):
        assert rel(a, r, 1e-12) < tol


@pytest.mark.parametrize("name", list(DRAWS))
def test_base_frame_forward_fp64(name):
    """The FP64 handles' forward step, in the base frame: end state and
    trajectory."""
    from paper_2109_07719_amd.sim import Sim
    b = synth.make_batch(DRAWS[name], 1e-3)
    print("case", name, flush=True)
    sim = Sim(b.systems, (1.0, -9.0, 2.0), dtype=torch.float64)
    f = lambda x: torch.tensor(np.ascontiguousarray(x), device="cuda")
    qT, qdT, tr = sim.forward(f(b.q0), f(b.qd0), f(b.tau), b.dt, K=0, traj=True)
    q1, qd1, _ = sim.forward(f(b.q0), f(b.qd0), f(b.tau[:1]), b.dt, K=0)
    oq, ov, ou = b.offsets()
    for k, s in enumerate(b.systems):
        m = O.Model(s, (1.0, -9.0, 2.0))
        q, v, u = slice(oq[k], oq[k + 1]), slice(ov[k], ov[k + 1]), slice(ou[k], ou[k + 1])
        tol = 1e-13 * max(s.n, 4) ** 3
        for a, r in zip((qT[q], qdT[v]), O.rollout(m, b.q0[q], b.qd0[v], b.tau[:, u], b.dt)):
            assert rel(a.cpu().numpy(), r, 1e-12) < tol, (k, s.n)
        for a, r in zip((q1[q], qd1[v]), O.rollout(m, b.q0[q], b.qd0[v], b.tau[:1, u], b.dt)):
            assert rel(a.cpu().numpy(), r, 1e-12) < tol, (k, s.n)
    row = tr.cpu().numpy()
    assert np.array_equal(row[0, :oq[-1]], q1.cpu().numpy()) and np.array_equal(row[-1, oq[-1]:], qdT.cpu().numpy())
