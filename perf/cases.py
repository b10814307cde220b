"""Timed cases of the framework's main paths, through its public entry points.

``listed()`` names the cases, ``draw(rng)`` draws further ones of the same
ranges, ``prepare`` builds what a program holds before the call (handle,
inputs), ``run`` makes one pass, ``work`` counts the bytes and operations the
pass cannot do without, and ``exact`` computes what ``run`` returns in 64
bits with plain torch: joint-space inertia matrix and bias forces from
masked sums over ancestor sets, a Cholesky solve, and autograd one step at a
time backwards.

A case is one of five kinds:
  rollout  sim.rollout forwards and backwards (one-step calls, checkpointed
           horizons, every system family), gradients of q0, qd0 and tau
  trajopt  TrajOpt.loss() and its backward pass: rollout, end-effector
           kinematics, loss
  jvp      Sim.forward_jvp, the forward-mode tangent
  contact  ContactBatch.rollout with its trajectory, then ContactBatch.grad
  pgs      pgs.pgs forwards and backwards
"""
import math

import numpy as np
import torch

from paper_2109_07719_amd import synth

DEV = "cuda"
GRAV = (0.0, -9.81, 0.0)
MU, BETA, SWEEPS = 0.8, 0.2, 30
REV, FREE, PRISM, BALL = 0, 1, 2, 3


def listed():
    return [
        # one environment, one step and its vector-Jacobian product: a policy
        # gradient step of a single robot, all latency
        dict(name="step_quad_1", kind="rollout", family="quad", B=1, lo=0, hi=0, T=1, K=1, dtype="f32"),
        # the same for a batch of samples (policy enhancement)
        dict(name="step_quad_4096", kind="rollout", family="quad", B=4096, lo=0, hi=0, T=1, K=1, dtype="f32"),
        # one 7-joint arm over a second in double precision
        dict(name="chain7_f64_1", kind="rollout", family="chain", B=1, lo=7, hi=7, T=1000, K=1, dtype="f64"),
        # the benchmark's batch of 7-joint arms, a shorter horizon
        dict(name="chain7_4096", kind="rollout", family="chain", B=4096, lo=7, hi=7, T=200, K=1, dtype="f32"),
        # the uneven branched trees of 6 to 40 links
        dict(name="trees_8192", kind="rollout", family="tree", B=8192, lo=6, hi=40, T=50, K=1, dtype="f32"),
        # free-floating quadrupeds, a checkpoint every tenth step
        dict(name="quads_1024_k10", kind="rollout", family="quad", B=1024, lo=0, hi=0, T=200, K=10, dtype="f32"),
        # quadrupeds on ball hips
        dict(name="ball_quads_1024", kind="rollout", family="ballquad", B=1024, lo=0, hi=0, T=100, K=1, dtype="f32"),
        # one trajectory-optimisation iteration on chains of 5 to 50 links
        dict(name="trajopt_2048", kind="trajopt", family="chain", B=2048, lo=5, hi=50, T=50, K=1, dtype="f32"),
        # tangents of short tree rollouts (sample enhancement)
        dict(name="jvp_trees_1000", kind="jvp", family="tree", B=1000, lo=6, hi=40, T=10, K=1, dtype="f32"),
        # quadrupeds standing on the ground: rollout with contact, its gradient
        dict(name="contact_4096", kind="contact", family="stand", B=4096, lo=0, hi=0, T=8, K=0, dtype="f32"),
        # a small batch of them over a longer horizon, in double precision
        dict(name="contact_f64_250", kind="contact", family="stand", B=250, lo=0, hi=0, T=60, K=0, dtype="f64"),
        # the batched contact solver: 12 rows (four contacts), 30 sweeps
        dict(name="pgs_12_32768", kind="pgs", family="mlcp", B=32768, lo=12, hi=12, T=30, K=0, dtype="f32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes over the listed ranges (logarithmic), odd ones
    among them, at most about the largest listed case's cost."""
    kind = rng.choice(["rollout"] * 5 + ["trajopt", "jvp", "contact", "contact", "pgs"])
    c = dict(kind=kind, family="mlcp", B=1, lo=0, hi=0, T=1, K=1, dtype="f64" if rng.random() < 0.25 else "f32")
    if kind == "pgs":
        c.update(B=_log(rng, 64, 30000), lo=rng.randint(3, 16), T=rng.randint(5, 50), K=0)
        c["hi"] = c["lo"]
    elif kind == "contact":
        c.update(family="stand", B=_log(rng, 16, 4000), T=_log(rng, 1, 8 if c["dtype"] == "f32" else 16), K=0)
    else:
        fam = "chain" if kind == "trajopt" else rng.choice(["chain", "tree", "ptree", "quad", "tquad", "ballquad"])
        c["family"] = fam
        lo, hi = {"chain": rng.choice([(7, 7), (2, 9), (5, 50)]), "tree": (6, 40), "ptree": (6, 40)}.get(fam, (0, 0))
        if kind == "trajopt":
            lo, hi = 5, rng.randint(20, 50)
        mean = {"chain": (lo + hi) / 2, "tree": 23, "ptree": 23}.get(fam, 18)
        steps = {"trajopt": 50, "jvp": 20}.get(kind, 200)
        c.update(lo=lo, hi=hi, T=_log(rng, 1, steps))
        most = 3.0e6 / (mean * c["T"])  # a third of the largest listed cases' DOF-steps
        c["B"] = max(1, _log(rng, 1, max(2, min(8000, most))))
        c["K"] = rng.choice([1, 1, 1, 7, 10]) if kind == "rollout" else 1
    return c


# ------------------------------------------------------------------- inputs
def _tree_parent(rng, n):
    """Breadth-first growth, 1 to 3 children a node, at most 6 levels."""
    while True:
        parent, depth, head = [-1], [1], 0
        while head < len(parent) and len(parent) < n:
            if depth[head] < 6:
                for _ in range(int(rng.integers(1, 4))):
                    if len(parent) < n:
                        parent.append(head)
                        depth.append(depth[head] + 1)
            head += 1
        if len(parent) == n:
            return np.array(parent, np.int32)


def _unit(x):
    return x / np.linalg.norm(x, axis=-1, keepdims=True)


QUAD_PARENT = np.array([-1] + [p for k in range(4) for p in (0, 3 * k + 1, 3 * k + 2)], np.int32)


def _inputs(case, seed):
    """Flat float64 arrays of the whole batch (rounded to the case's type)."""
    rng = np.random.default_rng([seed, case["B"], case["T"]])
    B, fam, lo, hi = case["B"], case["family"], case["lo"], case["hi"]
    topo, shape = [], np.random.default_rng([B, lo, hi])  # the structures go with the case, not the seed
    if fam == "chain":
        sizes = shape.integers(lo, hi + 1, B)
        topo = [np.arange(-1, n - 1, dtype=np.int32) for n in sizes]
    elif fam in ("tree", "ptree"):
        pool = [_tree_parent(shape, int(shape.integers(lo, hi + 1))) for _ in range(min(B, 512))]
        topo = [pool[k % len(pool)] for k in range(B)]
        sizes = np.array([len(p) for p in topo])
    else:
        sizes = np.full(B, 13)
        topo = [QUAD_PARENT] * B
    parent = np.concatenate(topo)
    off = np.concatenate([[0], np.cumsum(sizes)])
    N = int(off[-1])
    jtype = np.zeros(N, np.int32)
    rT, com, Ic, ET = np.zeros((N, 3)), np.zeros((N, 3)), np.zeros((N, 6)), np.tile(np.eye(3), (N, 1, 1))
    axis = np.tile([0.0, 0.0, 1.0], (N, 1))
    if fam in ("chain", "tree", "ptree"):
        mass = rng.uniform(0.5, 2.0, N)
        Ic[:, :3] = rng.uniform(0.01, 0.1, (N, 3))
        if fam == "chain":
            rT[parent >= 0, 0] = 0.5
            com[:, 0] = 0.25
        else:
            axis, rT = _unit(rng.normal(size=(N, 3))), 0.5 * _unit(rng.normal(size=(N, 3)))
            com = rng.uniform(-0.25, 0.25, (N, 3))
            if fam == "ptree":
                jtype[shape.random(N) < 0.3] = PRISM
    else:  # quadrupeds: box base on a free joint, legs hip x, thigh z, calf z
        loc = np.arange(N) % 13
        leg, part = (loc - 1) // 3, (loc - 1) % 3
        base = loc == 0
        mass = np.where(base, 10.0, rng.uniform(0.3, 1.5, N))
        Ic[:, :3] = np.where(base[:, None], 10.0 / 12 * np.array([0.1125, 0.45, 0.3825]), rng.uniform(0.001, 0.01, (N, 3)))
        hip, calf = ~base & (part == 0), ~base & (part == 2)
        rT[hip] = np.stack([0.25 * np.where(leg < 2, 1, -1), 0.0 * leg, 0.1 * np.where(leg % 2 == 0, 1, -1)], 1)[hip]
        rT[calf] = [0.0, -0.25, 0.0]
        com[~base & (part > 0)] = [0.0, -0.125, 0.0]
        axis[hip] = [1.0, 0.0, 0.0]
        jtype[base] = FREE
        if fam == "tquad":
            jtype[calf], axis[calf] = PRISM, [0.0, 1.0, 0.0]
        if fam == "ballquad":
            jtype[hip] = BALL
    nq, nv, nu = (np.select([jtype == FREE, jtype == BALL], v, 1) for v in ([7, 4], [6, 3], [0, 3]))
    qi, vi = np.cumsum(nq) - nq, np.cumsum(nv) - nv
    q, qd = rng.normal(0, 0.1, int(nq.sum())), rng.normal(0, 0.1, int(nv.sum()))
    tau = rng.normal(0, 0.3 if fam == "stand" else 1.0, (case["T"], int(nu.sum())))
    if case["kind"] == "trajopt":
        q[:], qd[:], tau[:] = 0, 0, 0.1 * tau
    fr, bl = np.nonzero(jtype == FREE)[0], np.nonzero(jtype == BALL)[0]
    if len(fr):
        q[qi[fr][:, None] + np.arange(3)] = rng.normal(0, 0.2, (len(fr), 3)) + [0, 0.5, 0]
        quat = rng.normal(size=(len(fr), 4))
        if fam == "stand":
            # crouched and sinking, so that the feet stay on the ground
            q[qi[fr][:, None] + np.arange(3)] = [0.0, 0.5, 0.0]
            quat = 0.02 * quat + [0, 0, 0, 1]
            q[qi[~base & (part == 1)]] += 0.6
            q[qi[calf]] -= 1.2
            qd[vi[fr] + 4] -= 0.5
            tau[:, 2::3] += 8.0  # the knees carry the weight
        q[qi[fr][:, None] + 3 + np.arange(4)] = _unit(quat)
    if len(bl):
        w = rng.normal(0, 0.3, (len(bl), 3))
        th = np.linalg.norm(w, axis=1, keepdims=True)
        q[qi[bl][:, None] + np.arange(4)] = np.concatenate([np.sin(th / 2) * w / th, np.cos(th / 2)], 1)
    r = (lambda x: np.asarray(x, np.float32).astype(np.float64)) if case["dtype"] == "f32" else (lambda x: x)
    d = dict(parent=parent, jtype=jtype, off=off, nq=nq, nv=nv, nu=nu, qi=qi, vi=vi, E_T=r(ET), r_T=r(rT), axis=r(axis),
             mass=r(mass), com=r(com), Ic=r(Ic), q=r(q), qd=r(qd), tau=r(tau), g=r(np.array(GRAV)),
             dt=float(r(5e-4 if fam in ("tree", "ptree") else 1e-3)))
    d["gq"], d["gqd"] = r(rng.normal(size=q.shape)), r(rng.normal(size=qd.shape))
    if case["kind"] == "trajopt":
        phi = rng.uniform(-math.pi, math.pi, (B, 2))  # targets within reach of every chain
        reach = 0.5 * sizes * rng.uniform(0.2, 0.9, B)
        d["target"] = r(np.stack([reach * np.cos(phi[:, 0]), reach * np.sin(phi[:, 0]), 0 * reach], 1))
    if case["kind"] == "jvp":
        d["dq"], d["dqd"], d["dtau"] = (r(rng.normal(size=x.shape)) for x in (q, qd, tau))
    if case["kind"] == "contact":
        # the feet stand 0.15 to 0.4 mm deep, one in four is lifted by two to three centimetres:
        # the sphere's radius is its centre's height plus the depth
        depth = np.where(rng.random((B, 4)) < 0.25, -rng.uniform(0.02, 0.03, (B, 4)), rng.uniform(1.5e-4, 4e-4, (B, 4)))
        m = Model(d, "cpu")
        R, p = m.poses(torch.tensor(d["q"]))
        foot = p[:, 3::3] + (R[:, 3::3] @ torch.tensor([0.0, -0.25, 0.0], dtype=torch.float64))
        Rw, pw = m.base(torch.tensor(d["q"]))
        y = (pw[:, None] + foot @ Rw.transpose(1, 2))[..., 1].numpy()
        d["centers"], d["radii"] = r(np.tile([0.0, -0.25, 0.0], (B, 4, 1))), r(np.maximum(y + depth, 0.01))
    return d


def _mlcp(case, seed):
    """Delassus-like problems, diagonally dominant rows, boxes, some one-sided."""
    dt = torch.float64
    g = torch.Generator(device=DEV).manual_seed(seed * 7 + 3)
    B, n = case["B"], case["lo"]
    f = lambda *s: torch.randn(s, generator=g, device=DEV, dtype=dt)
    u = lambda *s: torch.rand(s, generator=g, device=DEV, dtype=dt)
    G = f(B, n, n)
    A = (G @ G.transpose(1, 2).contiguous()) / n + 0.05 * f(B, n, n)
    A = A + torch.diag_embed(1.0 + A.abs().sum(-1) * 0.3)
    half = 0.05 + 0.55 * u(B, n)
    one = u(B, n) < 0.3
    lo, hi = torch.where(one, torch.zeros_like(half), -half), torch.where(one, torch.full_like(half, 3e38), half)
    out = [A, 1.5 * f(B, n), lo, hi, 0.3 * f(B, n), f(B, n)]
    return [x.float() for x in out] if case["dtype"] == "f32" else out


def _dtype(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


def _systems(d):
    o = d["off"]
    return [synth.System(*(d[k][a:b] for k in ("parent", "jtype", "E_T", "r_T", "axis", "mass", "com", "Ic")))
            for a, b in zip(o[:-1], o[1:])]


def prepare(case, seed):
    dt = _dtype(case)
    if case["kind"] == "pgs":
        A, b, lo, hi, x0, xb = _mlcp(case, seed)
        return dict(case=case, leaves=[x.requires_grad_() for x in (A, b, lo, hi, x0)], xb=xb)
    d = _inputs(case, seed)
    f = lambda x: torch.tensor(np.ascontiguousarray(x), dtype=dt, device=DEV)
    s = dict(case=case, dt=d["dt"])
    systems = _systems(d)
    if case["kind"] == "contact":
        from paper_2109_07719_amd.contact import ContactBatch
        B, bm = case["B"], lambda x: f(x.reshape(*x.shape[:-1], case["B"], -1).swapaxes(-1, -2))
        s["cb"] = ContactBatch(systems, [3, 6, 9, 12], d["centers"], d["radii"], mu=MU, beta=BETA, niter=SWEEPS,
                               gravity=GRAV, dtype=dt)
        s.update({k: bm(d[k]) for k in ("q", "qd", "tau", "gq", "gqd")})
        return s
    if case["kind"] == "trajopt":
        from paper_2109_07719_amd.trajopt import TrajOpt
        batch = synth.Batch(systems=systems, q0=d["q"], qd0=d["qd"], tau=d["tau"], dt=d["dt"], gravity=d["g"])
        s["opt"] = TrajOpt(batch, d["target"], [x.n - 1 for x in systems], np.tile([0.5, 0.0, 0.0], (len(systems), 1)),
                           K=case["K"], dtype=dt)
        return s
    from paper_2109_07719_amd.sim import Sim
    s["sim"] = Sim(systems, GRAV, dtype=dt)
    s.update({k: f(d[k]) for k in ("q", "qd", "tau", "gq", "gqd", "dq", "dqd", "dtau") if k in d})
    if case["kind"] == "rollout":
        for k in ("q", "qd", "tau"):
            s[k].requires_grad_()
    return s


def run(state):
    s, kind = state, state["case"]["kind"]
    if kind == "rollout":
        from paper_2109_07719_amd.sim import rollout
        x = (s["q"], s["qd"], s["tau"])
        y = rollout(s["sim"], *x, s["dt"], K=s["case"]["K"])
        return [v.detach() for v in y] + list(torch.autograd.grad(y, x, (s["gq"], s["gqd"])))
    if kind == "trajopt":
        opt = s["opt"]
        opt.opt.zero_grad(set_to_none=False)
        loss, per = opt.loss()
        loss.backward()
        return [loss.detach(), per.detach(), opt.tau.grad]
    if kind == "jvp":
        return list(s["sim"].forward_jvp(s["q"], s["qd"], s["tau"], s["dq"], s["dqd"], s["dtau"], s["dt"]))
    if kind == "contact":
        cb = s["cb"]
        qT, qdT, tr = cb.rollout(s["q"], s["qd"], s["tau"], s["dt"])
        return [qT, qdT] + list(cb.grad(tr, s["tau"], s["dt"], s["gq"], s["gqd"]))
    from paper_2109_07719_amd.pgs import pgs
    x = pgs(*s["leaves"], s["case"]["T"])
    return [x.detach()] + list(torch.autograd.grad(x, s["leaves"], s["xb"]))


def work(case):
    """Inputs read once, outputs written once; operations of the recursive
    algorithms: about 420 (z-aligned chains) to 660 a degree of freedom and
    step forwards, three times that with the adjoint."""
    es = 8 if case["dtype"] == "f64" else 4
    B, T, n = case["B"], case["T"], (case["lo"] + case["hi"]) / 2
    if case["kind"] == "pgs":
        n = case["lo"]
        return dict(bytes=es * B * (2 * n * n + 10 * n), flops=B * T * (8.0 * n * n))
    nq, nv, nu = {"quad": (19, 18, 12), "tquad": (19, 18, 12), "stand": (19, 18, 12),
                  "ballquad": (31, 26, 20)}.get(case["family"], (n, n, n))
    par = B * es * 25 * (13 if case["lo"] == 0 else n)
    per = 420.0 if case["family"] == "chain" else 660.0
    if case["kind"] == "contact":
        # per step and system: the smooth step and its adjoint, twelve solves with
        # the inertia matrix and their adjoints, two solves of 30 sweeps and theirs
        return dict(bytes=par + es * B * (3 * (nq + nv) + T * (2 * nu + nq + nv)),
                    flops=B * T * (3 * per * nv + 12 * 60.0 * nv * 2 + 2 * SWEEPS * 12 * 24 * 3.0))
    state = es * B * (nq + nv)
    if case["kind"] == "jvp":
        return dict(bytes=par + 4 * state + 2 * es * B * T * nu, flops=2.5 * per * B * nv * T)
    return dict(bytes=par + 4 * state + 2 * es * B * T * nu, flops=3.0 * per * B * nv * T)


# -------------------------------------------------------- the same in 64 bits
def _cross(a, b):
    return torch.linalg.cross(a, b, dim=-1)


def _rot(qt):
    """R = (w^2 - u.u) 1 + 2 u u^T + 2 w [u]x of a quaternion (u, w)."""
    x, y, z, w = qt.unbind(-1)
    d = w * w - x * x - y * y - z * z
    rows = [d + 2 * x * x, 2 * (x * y - w * z), 2 * (x * z + w * y), 2 * (x * y + w * z), d + 2 * y * y,
            2 * (y * z - w * x), 2 * (x * z - w * y), 2 * (y * z + w * x), d + 2 * z * z]
    return torch.stack(rows, -1).reshape(*qt.shape[:-1], 3, 3)


def _quat_step(qt, w1, dt):
    u, s = qt[..., :3], qt[..., 3:]
    r = qt + 0.5 * dt * torch.cat([s * w1 + _cross(u, w1), -(u * w1).sum(-1, keepdim=True)], -1)
    return r / r.norm(dim=-1, keepdim=True)


class Model:
    """A batch padded to the largest system; coordinates are those of the
    base (of the free root's own frame where there is one)."""

    def __init__(self, d, dev=DEV):
        f = lambda x: torch.tensor(np.ascontiguousarray(x), dtype=torch.float64, device=dev)
        i64 = lambda x: torch.tensor(np.ascontiguousarray(x), dtype=torch.long, device=dev)
        off, par, jt = d["off"], d["parent"], d["jtype"]
        B, N = len(off) - 1, len(par)
        self.B, self.n, self.dt, self.N = B, int(np.diff(off).max()), d["dt"], N
        sysof = np.repeat(np.arange(B), np.diff(off))
        loc = np.arange(N) - off[sysof]
        gpar = np.where(par >= 0, off[sysof] + par, -1)
        depth = np.zeros(N, int)
        for k in range(1, self.n):
            at = np.nonzero((loc == k) & (par >= 0))[0]
            depth[at] = depth[gpar[at]] + 1
        self.levels = [(i64(a), i64(np.maximum(gpar[a], 0)), bool(k == 0))
                       for k in range(depth.max() + 1) for a in [np.nonzero(depth == k)[0]]]
        self.slot = i64(sysof * self.n + loc)  # link -> padded place
        # degrees of freedom, in the order of qd
        link = np.repeat(np.arange(N), d["nv"])
        nv_sys = np.add.reduceat(d["nv"], off[:-1])
        v0 = np.concatenate([[0], np.cumsum(nv_sys)])
        self.nv, dsys = int(nv_sys.max()), sysof[link]
        dloc = np.arange(len(link)) - v0[dsys]
        k = np.arange(len(link)) - d["vi"][link]
        ax = _unit(d["axis"])[link]
        multi = (jt[link] == FREE) | (jt[link] == BALL)
        ax[multi] = np.eye(3)[k[multi] % 3]
        self.dax, self.dlink = f(ax), i64(link)
        self.dang = f(((jt[link] == REV) | (multi & (k < 3))).astype(float))[:, None]
        self.dslot = i64(dsys * self.nv + dloc)
        act = jt[link] != FREE
        self.act = i64((dsys * self.nv + dloc)[act])
        anc = np.zeros((B, self.n, self.n), bool)  # anc[b, i, j]: j on i's path to the root
        for kk in range(self.n):
            at = np.nonzero(loc == kk)[0]
            ch = at[par[at] >= 0]
            anc[sysof[ch], kk] = anc[sysof[ch], par[ch]]
            anc[sysof[at], kk, kk] = True
        dl = np.full((B, self.nv), 0)
        used = np.zeros((B, self.nv), bool)
        dl[dsys, dloc], used[dsys, dloc] = loc[link], True
        take = np.take_along_axis(anc, dl[:, None, :], 2) & used[:, None, :]  # [B, n, nv]
        self.path = f(take)
        self.dl = i64(dl)
        mk = np.take_along_axis(take, dl[:, :, None], 1) & used[:, :, None]  # k's link below l's
        self.low = f(mk)
        self.strict = f(mk & ~np.swapaxes(mk, 1, 2))
        self.pad = torch.diag_embed(f(~used))
        self.sub = f(anc).transpose(1, 2).contiguous()  # subtree sums
        self.ET, self.rT, self.ax = f(d["E_T"]).transpose(1, 2).contiguous(), f(d["r_T"]), f(_unit(d["axis"]))
        a = self.ax
        z = torch.zeros_like(a[:, 0])
        self.K = torch.stack([z, -a[:, 2], a[:, 1], a[:, 2], z, -a[:, 0], -a[:, 1], a[:, 0], z], 1).reshape(-1, 3, 3)
        self.mass, self.com = f(d["mass"]), f(d["com"])
        I = d["Ic"]
        self.Ic = f(I[:, [0, 3, 4, 3, 1, 5, 4, 5, 2]].reshape(-1, 3, 3))
        qi, vi = d["qi"], d["vi"]
        self.rev, self.pri = f(jt == REV)[:, None, None], f(jt == PRISM)[:, None]
        self.q1 = i64(qi)
        one = np.nonzero((jt == REV) | (jt == PRISM))[0]
        fr, bl = np.nonzero(jt == FREE)[0], np.nonzero(jt == BALL)[0]
        self.oq, self.ov = i64(qi[one]), i64(vi[one])
        self.fr, self.frq, self.frv = len(fr), i64(qi[fr][:, None] + np.arange(7)), i64(vi[fr][:, None] + np.arange(6))
        self.bl, self.blq, self.blv = i64(bl), i64(qi[bl][:, None] + np.arange(4)), i64(vi[bl][:, None] + np.arange(3))
        self.frl = i64(fr)
        self.g = f(d["g"])

    def base(self, q):
        """World rotation and position of the base frame, per system."""
        if not self.fr:
            return None, None
        x = q[self.frq]
        return _rot(x[:, 3:]), x[:, :3]

    def poses(self, q, flat=False):
        """Link rotations and origins in the base frame."""
        qj = q[self.q1]
        s, c = torch.sin(qj)[:, None, None], torch.cos(qj)[:, None, None]
        I3 = torch.eye(3, dtype=q.dtype, device=q.device)
        Rl = self.ET @ (I3 + self.rev * (s * self.K + (1 - c) * (self.K @ self.K)))
        pl = self.rT + (self.ET @ (self.pri * qj[:, None] * self.ax)[..., None])[..., 0]
        if self.bl.numel():
            Rl = Rl.index_copy(0, self.bl, self.ET[self.bl] @ _rot(q[self.blq]))
        if self.fr:
            Rl = Rl.index_copy(0, self.frl, I3.expand(self.fr, 3, 3))
            pl = pl.index_copy(0, self.frl, torch.zeros(self.fr, 3, dtype=q.dtype, device=q.device))
        R, p = Rl, pl
        for idx, par, root in self.levels:
            if root:
                continue
            Rp = R[par]
            p = p.index_copy(0, idx, p[par] + (Rp @ pl[idx][..., None])[..., 0])
            R = R.index_copy(0, idx, Rp @ Rl[idx])
        if flat:
            return R, p
        return self._pad(R, self.slot, self.n), self._pad(p, self.slot, self.n)

    def _pad(self, x, slot, m):
        out = torch.zeros(self.B * m, *x.shape[1:], dtype=x.dtype, device=x.device)
        return out.index_copy(0, slot, x).reshape(self.B, m, *x.shape[1:])

    def dynamics(self, q, qd):
        """M and the bias (M qdd = u - bias), and the links' poses."""
        R, p = self.poses(q, flat=True)
        a = (R[self.dlink] @ self.dax[..., None])[..., 0]
        ang = self.dang * a
        lin = (1 - self.dang) * a + _cross(p[self.dlink], ang)
        S = self._pad(torch.cat([ang, lin], 1), self.dslot, self.nv)
        w = S * self._pad(qd[:, None], self.dslot, self.nv)
        V = self.path @ w
        Vk = torch.gather(V, 1, self.dl[..., None].expand(-1, -1, 6))
        c = torch.cat([_cross(Vk[..., :3], w[..., :3]),
                       _cross(Vk[..., 3:], w[..., :3]) + _cross(Vk[..., :3], w[..., 3:])], -1)
        g = self.g.expand(self.B, 3)
        if self.fr:
            g = (self.base(q)[0].transpose(1, 2) @ self.g)
        A = self.path @ c - torch.cat([torch.zeros_like(g), g], -1)[:, None]
        # inertias about the frame's origin: mass, first moment, second moment
        cw = p + (R @ self.com[..., None])[..., 0]
        mc = self.mass[:, None] * cw
        I3 = torch.eye(3, dtype=q.dtype, device=q.device)
        IO = R @ self.Ic @ R.transpose(1, 2) + self.mass[:, None, None] * (
            (cw * cw).sum(-1)[:, None, None] * I3 - cw[:, :, None] * cw[:, None, :])
        J = self._pad(torch.cat([self.mass[:, None], mc, IO.reshape(-1, 9)], 1), self.slot, self.n)

        def mul(J, x):
            m, mc, I = J[..., :1], J[..., 1:4], J[..., 4:].reshape(*J.shape[:-1], 3, 3)
            return torch.cat([(I @ x[..., :3, None])[..., 0] + _cross(mc, x[..., 3:]),
                              m * x[..., 3:] - _cross(mc, x[..., :3])], -1)
        h = mul(J, V)
        f = mul(J, A) + torch.cat([_cross(V[..., :3], h[..., :3]) + _cross(V[..., 3:], h[..., 3:]),
                                   _cross(V[..., :3], h[..., 3:])], -1)
        F = self.path.transpose(1, 2) @ f
        bias = (S * F).sum(-1)
        Jc = torch.gather(self.sub @ J, 1, self.dl[..., None].expand(-1, -1, 13))
        G = mul(Jc, S) @ S.transpose(1, 2).contiguous()
        M = G * self.low + (G * self.strict).transpose(1, 2) + self.pad
        return M, bias, R, p

    def step(self, q, qd, u, contact=None):
        M, bias, R, p = self.dynamics(q, qd)
        tau = torch.zeros(self.B * self.nv, dtype=q.dtype, device=q.device).index_copy(0, self.act, u)
        L = torch.linalg.cholesky(M)
        acc = torch.cholesky_solve((tau.reshape(self.B, self.nv) - bias)[..., None], L)[..., 0]
        qd1 = qd + self.dt * acc.reshape(-1)[self.dslot]
        if contact is not None:
            qd1 = qd1 + contact(self, q, qd1, L, R, p).reshape(-1)[self.dslot]
        q1 = q.index_copy(0, self.oq, q[self.oq] + self.dt * qd1[self.ov])
        if self.fr:
            x, v = q[self.frq], qd1[self.frv]
            pn = x[:, :3] + self.dt * (_rot(x[:, 3:]) @ v[:, 3:, None])[..., 0]
            q1 = q1.index_copy(0, self.frq.reshape(-1), torch.cat([pn, _quat_step(x[:, 3:], v[:, :3], self.dt)], 1).reshape(-1))
        if self.bl.numel():
            q1 = q1.index_copy(0, self.blq.reshape(-1), _quat_step(q[self.blq], qd1[self.blv], self.dt).reshape(-1))
        return q1, qd1


def _sweeps(A, b, lo, hi, x, keep, niter):
    """Projected Gauss-Seidel sweeps; rows not kept stay zero."""
    n = b.shape[-1]
    x, diag = list(x.unbind(-1)), torch.diagonal(A, dim1=-2, dim2=-1)
    off = A - torch.diag_embed(diag)
    if keep is not None:
        diag = torch.where(keep, diag, torch.ones_like(diag))
    for _ in range(niter):
        for i in range(n):
            y = -(b[:, i] + (off[:, i] * torch.stack(x, -1)).sum(-1)) / diag[:, i]
            y = torch.where(y < lo[:, i], lo[:, i], torch.where(y > hi[:, i], hi[:, i], y))
            x[i] = y if keep is None else torch.where(keep[:, i], y, torch.zeros_like(y))
    return torch.stack(x, -1)


def _contact(d, dev=DEV):
    f = lambda x: torch.tensor(np.ascontiguousarray(x), dtype=torch.float64, device=dev)
    cen, rad = f(d["centers"]), f(d["radii"])
    f32 = not np.array_equal(np.array(MU), np.float32(MU)) and np.array_equal(d["mass"], d["mass"].astype(np.float32))
    mu, beta = (float(np.float32(MU)), float(np.float32(BETA))) if f32 else (MU, BETA)

    def resolve(m, q, qdm, L, R, p):
        Rw, pw = m.base(q)
        a = m._pad((R[m.dlink] @ m.dax[..., None])[..., 0], m.dslot, m.nv) @ Rw.transpose(1, 2)
        at, ang = m._pad(p[m.dlink], m.dslot, m.nv), m._pad(m.dang, m.dslot, m.nv)[:, None]
        R, p = (m._pad(x, m.slot, m.n)[:, 3::3] for x in (R, p))
        up = Rw[:, 1][:, None]  # the world's y axis in the base frame
        cb = p + (R @ cen[..., None])[..., 0]
        phi = pw[:, None, 1] + (cb * up).sum(-1) - rad
        pt = cb - rad[..., None] * up
        path = m.path[:, 3::3]  # [B, 4, nv]
        # world velocity of the point: axis x arm, both turned into the world (the
        # reading of R off the unit sphere that the gradient's radial part goes by)
        arm = (pt[:, :, None] - at[:, None]) @ Rw.transpose(1, 2)[:, None]
        a4 = a[:, None].expand(-1, 4, -1, -1)
        v = path[..., None] * (ang * _cross(a4, arm) + (1 - ang) * a4)
        J = v[..., [1, 0, 2]].transpose(2, 3).reshape(m.B, 12, m.nv)
        on = (phi < 0).repeat_interleave(3, 1)
        J = J * on[..., None]
        W = torch.cholesky_solve(J.transpose(1, 2).contiguous(), L)
        A = J @ W
        n = torch.arange(12, device=q.device) % 3 == 0
        b = (J @ m._pad(qdm, m.dslot, m.nv)[..., None])[..., 0] + torch.where(
            n & on, (beta / m.dt) * phi.repeat_interleave(3, 1), torch.zeros_like(on, dtype=q.dtype))
        diag = torch.diagonal(A, dim1=1, dim2=2)
        keep = on & (diag > 1e-12 * diag.amax(1, keepdim=True))
        z, big = torch.zeros_like(b), torch.full_like(b, 1e30)
        l1 = _sweeps(A[:, ::3, ::3], b[:, ::3], z[:, ::3], big[:, ::3], z[:, ::3], keep[:, ::3], SWEEPS)
        lim = mu * l1.repeat_interleave(3, 1)
        lam = _sweeps(A, b, torch.where(n, z, -lim), torch.where(n, big, lim), z, keep, SWEEPS)
        return (W @ lam[..., None])[..., 0]
    return resolve


def exact(case, seed):
    if case["kind"] == "pgs":
        A, b, lo, hi, x0, xb = (x.detach().double() for x in _mlcp(case, seed))
        x = [v.requires_grad_() for v in (A, b, lo, hi, x0)]
        y = _sweeps(*x, None, case["T"])
        return [y.detach()] + list(torch.autograd.grad(y, x, xb))
    if case["T"] * (case["hi"] + 20) > 60000:
        return None  # minutes of small operations
    d = _inputs(case, seed)
    m = Model(d)
    f = lambda x: torch.tensor(np.ascontiguousarray(x), dtype=torch.float64, device=DEV)
    q, qd, tau, T = f(d["q"]), f(d["qd"]), f(d["tau"]), case["T"]
    if case["kind"] == "jvp":
        import torch.autograd.forward_ad as fa
        with fa.dual_level():
            x = [fa.make_dual(q, f(d["dq"])), fa.make_dual(qd, f(d["dqd"]))]
            u = fa.make_dual(tau, f(d["dtau"]))
            for t in range(T):
                x = m.step(*x, u[t])
            (q1, dq), (qd1, dqd) = (fa.unpack_dual(v) for v in x)
            return [q1.clone(), qd1.clone(), dq.clone(), dqd.clone()]
    contact = _contact(d) if case["kind"] == "contact" else None
    states = [(q, qd)]
    with torch.no_grad():
        for t in range(T):
            states.append(m.step(*states[-1], tau[t], contact))
    qT, qdT = states[-1]
    if case["kind"] == "trajopt":
        qT = qT.clone().requires_grad_()
        R, p = m.poses(qT, flat=True)
        last = torch.tensor(d["off"][1:] - 1, device=DEV)
        ee = p[last] + 0.5 * R[last][..., 0]
        per = ((ee - f(d["target"])) ** 2).sum(-1)
        gq, gqd = torch.autograd.grad(per.sum(), qT)[0], torch.zeros_like(qdT)
    else:
        gq, gqd = f(d["gq"]), f(d["gqd"])
    gtau = torch.empty_like(tau)
    for t in reversed(range(T)):
        x = [v.detach().requires_grad_() for v in (*states[t], tau[t])]
        gq, gqd, gtau[t] = torch.autograd.grad(m.step(*x, contact), x, (gq, gqd))
    if case["kind"] == "trajopt":
        w = 1e-4
        return [per.detach().sum() + w * (tau ** 2).sum(), per.detach(), gtau + 2 * w * tau]
    if m.bl.numel():  # the library returns a ball joint's gradient along the unit sphere
        n = _unit_t(q[m.blq])
        gb = gq[m.blq]
        gq = gq.index_copy(0, m.blq.reshape(-1), (gb - (gb * n).sum(-1, keepdim=True) * n).reshape(-1))
    if case["kind"] == "contact":
        bm = lambda x: x.reshape(*x.shape[:-1], m.B, -1).transpose(-1, -2).contiguous()
        return [bm(x) for x in (qT, qdT, gq, gqd, gtau)]
    return [qT, qdT, gq, gqd, gtau]


def _unit_t(x):
    return x / x.norm(dim=-1, keepdim=True)
