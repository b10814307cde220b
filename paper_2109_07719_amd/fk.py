"""Forward kinematics of link points in torch (loss-side helper).

Losses on the end state of a rollout (for example an end-effector target)
are ordinary differentiable torch code; their gradient with respect to q^T
becomes the seed of the adjoint pass (Sec. 3, Eq. diff_u: dPhi/dx^T enters
the adjoint recursion).  This module computes world positions of chosen
points on chosen links for a whole batch, one tree level at a time, with the
package's joint convention (revolute: link -> parent rotation
E^T = E_T^T Rot(a, q), Rot the rotation by +q about a, origin at r_T;
prismatic: E^T = E_T^T, origin at r_T + q E_T^T a; spherical: E^T =
E_T^T R(quat), origin at r_T; free root: R(quat) and p).  Other joint types
are rejected.

On the GPU the positions and their adjoint come from one kernel each
(`sim_link_points`), a point's path to the root composed by one wavefront;
anything beyond a plain first-order call (CPU tensors, higher derivatives,
forward mode, function transforms, batched cotangents, tracing) and points
whose paths share a link run the torch expressions.
"""
from __future__ import annotations

import numpy as np
import torch
import torch.autograd.forward_ad as fwad
from torch.utils._python_dispatch import _get_current_dispatch_mode

from . import _native as N
from .sim import _ptr, _stream

_DT = {torch.float32: N.SIM_F32, torch.float64: N.SIM_F64}
_MAX_PATH = 64   # one lane per link of a path


def _skew(a):
    z = torch.zeros_like(a[..., 0])
    return torch.stack([torch.stack([z, -a[..., 2], a[..., 1]], -1),
                        torch.stack([a[..., 2], z, -a[..., 0]], -1),
                        torch.stack([-a[..., 1], a[..., 0], z], -1)], -2)


def _quat_R(qt):
    x, y, z, w = qt.unbind(-1)
    return torch.stack([
        torch.stack([w * w + x * x - y * y - z * z, 2 * (x * y - w * z), 2 * (x * z + w * y)], -1),
        torch.stack([2 * (x * y + w * z), w * w - x * x + y * y - z * z, 2 * (y * z - w * x)], -1),
        torch.stack([2 * (x * z - w * y), 2 * (y * z + w * x), w * w - x * x - y * y + z * z], -1)], -2)


def _paths(target, parent, jtype, most=_MAX_PATH):
    """Links from the root to each target [n, longest], -1 past the end; a
    free link starts its path.  None where a path is too long or a target
    does not exist."""
    n = len(parent)
    if ((target < -n) | (target >= n)).any():
        return None
    cur, rows = np.where(target < 0, target + n, target), []
    while (cur >= 0).any():
        if len(rows) == most:
            return None
        rows.append(cur)
        up = np.where(cur >= 0, parent[cur], -1)
        cur = np.where((cur >= 0) & (jtype[cur] == 1), -1, up)
    up = np.stack(rows, axis=1)                      # target first
    size = (up >= 0).sum(axis=1, keepdims=True)
    k = size - 1 - np.arange(up.shape[1])[None]
    return np.where(k >= 0, np.take_along_axis(up, np.maximum(k, 0), axis=1), -1).astype(np.int32)


def _plain(t):
    """Whether t is an ordinary tensor outside every transform: one whose data
    a kernel may read."""
    if type(t) not in (torch.Tensor, torch.nn.Parameter):
        return False
    if torch.compiler.is_compiling() or torch.jit.is_tracing():
        return False
    F = torch._C._functorch
    if F.peek_interpreter_stack() is not None or _get_current_dispatch_mode() is not None:
        return False
    # cotangents of is_grads_batched and jacobian(vectorize=True) come without an interpreter
    return not F.is_legacy_batchedtensor(t) and fwad.unpack_dual(t).tangent is None


class _Points(torch.autograd.Function):
    @staticmethod
    def forward(ctx, q, fk):
        ctx.fk = fk
        ctx.save_for_backward(q, fk.ETt, fk.rT, fk.ax, fk.pts)
        x = torch.empty_like(fk.pts)
        fk._call("sim_link_points", q, fk.ETt, fk.rT, fk.ax, fk.pts, x)
        return x

    @staticmethod
    def backward(ctx, g):
        q, *tables = ctx.saved_tensors
        if torch.is_grad_enabled():   # a graph of the gradient is wanted
            return torch.autograd.grad(ctx.fk._positions(q), q, g, create_graph=True)[0], None
        if not _plain(g):
            with torch.enable_grad():
                v = q.detach().requires_grad_()
                x = ctx.fk._positions(v)
            return torch.autograd.grad(x, v, g)[0], None
        gq = torch.zeros_like(q)
        ctx.fk._call("sim_link_points_adjoint", q, *tables, g.contiguous(), gq)
        return gq, None


class LinkPoints(torch.nn.Module):
    """World positions of one point per system: point `pts[s]` (link
    coordinates) on link `links[s]` (local index) of system s."""

    _path = None   # the points' paths on the GPU, if the kernels take them

    def __init__(self, systems, links, pts, dtype=torch.float32, device="cuda"):
        super().__init__()
        glob_par, dep, qidx, jt, ET, rT, ax, target = [], [], [], [], [], [], [], []
        base, qbase = 0, 0
        for s, sy in enumerate(systems):
            d = sy.depth()
            qo = 0
            for i in range(sy.n):
                if int(sy.jtype[i]) not in (0, 1, 2, 3):
                    raise ValueError(f"LinkPoints: system {s} link {i} has joint type {int(sy.jtype[i])}; "
                                     "only revolute (0), free root (1), prismatic (2) and spherical (3) "
                                     "joints are supported")
                glob_par.append(-1 if sy.parent[i] < 0 else base + int(sy.parent[i]))
                dep.append(int(d[i]))
                qidx.append(qbase + qo)
                jt.append(int(sy.jtype[i]))
                ET.append(np.asarray(sy.E_T[i]))
                rT.append(np.asarray(sy.r_T[i]))
                ax.append(np.asarray(sy.axis[i]))
                qo += 7 if sy.jtype[i] == 1 else 4 if sy.jtype[i] == 3 else 1
            target.append(base + int(links[s]))
            base += sy.n
            qbase += qo
        f = lambda x: torch.tensor(np.asarray(x), dtype=dtype, device=device)
        i64 = lambda x: torch.tensor(np.asarray(x), dtype=torch.long, device=device)
        self.n_links = base
        self.parent = i64(glob_par)
        self.depth = np.asarray(dep)
        self.qidx = i64(qidx)
        self.qidx_np = np.asarray(qidx)
        self.jtype = np.asarray(jt)
        self.ETt = f(np.stack(ET)).transpose(-1, -2).contiguous()
        self.rT = f(np.stack(rT))
        self.K = _skew(f(np.stack(ax)))
        self.ax = f(np.stack(ax))
        self.prism = torch.tensor(np.asarray(jt) == 2, device=device)
        self.target = i64(target)
        self.pts = f(np.asarray(pts))
        self.levels = [torch.tensor(np.nonzero(self.depth == d)[0], dtype=torch.long, device=device)
                       for d in range(int(self.depth.max()) + 1)]
        self.level_free = [np.nonzero(self.jtype[np.nonzero(self.depth == d)[0]] == 1)[0]
                           for d in range(int(self.depth.max()) + 1)]
        self.level_ball = [np.nonzero(self.jtype[np.nonzero(self.depth == d)[0]] == 3)[0]
                           for d in range(int(self.depth.max()) + 1)]

        path = _paths(np.asarray(target), np.asarray(glob_par), self.jtype)
        # the adjoint kernel writes each path's joints: no two may share one
        on = [] if path is None else path[path >= 0]
        if path is not None and np.unique(on).size == on.size and self.rT.is_cuda:
            self._path = torch.tensor(path, device=device)
            self._jtype = torch.tensor(self.jtype, dtype=torch.int32, device=device)
            self._nq = int(qbase)

    def _native(self, q):
        """Whether a call on q is one the kernels take."""
        if self._path is None or q.dtype not in _DT or not _plain(q) or torch.is_autocast_enabled():
            return False
        fits = lambda t, n: (type(t) is torch.Tensor and t.dtype == q.dtype and t.device == q.device
                             and t.numel() == n and t.is_contiguous() and not t.requires_grad)
        n = self.n_links
        return (q.device == self._path.device and q.dim() == 1 and q.numel() >= self._nq and q.is_contiguous()
                and fits(self.ETt, 9 * n) and fits(self.rT, 3 * n) and fits(self.ax, 3 * n)
                and fits(self.pts, 3 * self._path.shape[0]) and self.pts.dim() == 2)

    def _call(self, name, q, ETt, rT, ax, pts, *last):
        p = _ptr
        with torch.cuda.device(q.device):
            N.check(getattr(N.lib(), name)(_DT[q.dtype], self._path.shape[0], self._path.shape[1], p(self._path),
                                           p(self._jtype), p(self.qidx), p(ETt), p(rT), p(ax), p(pts), p(q),
                                           *(p(t) for t in last), _stream()))

    def forward(self, q):
        if not self._native(q):
            return self._positions(q)
        # a copy for the adjoint: q may be changed in place after the call
        return _Points.apply(q.clone() if q.requires_grad and torch.is_grad_enabled() else q, self)

    def _positions(self, q):
        n = self.n_links
        Rw = torch.zeros((n, 3, 3), dtype=q.dtype, device=q.device)
        pw = torch.zeros((n, 3), dtype=q.dtype, device=q.device)
        I3 = torch.eye(3, dtype=q.dtype, device=q.device)
        for idx, free, ball in zip(self.levels, self.level_free, self.level_ball):
            m = idx.numel()
            qi = q[self.qidx[idx]]
            K = self.K[idx]
            pr = self.prism[idx]
            s, c = torch.sin(qi)[:, None, None], torch.cos(qi)[:, None, None]
            Rj = torch.where(pr[:, None, None], I3.expand(m, 3, 3), I3 + s * K + (1 - c) * (K @ K))
            if len(ball):
                rows = list(Rj.unbind(0))
                for k in ball:
                    qo = int(self.qidx_np[int(idx[k])])
                    rows[k] = _quat_R(q[qo:qo + 4])
                Rj = torch.stack(rows)
            par = self.parent[idx]
            has_par = par >= 0
            parc = par.clamp(min=0)
            Rp = torch.where(has_par[:, None, None], Rw[parc], I3.expand(m, 3, 3))
            pp = torch.where(has_par[:, None], pw[parc], torch.zeros((m, 3), dtype=q.dtype, device=q.device))
            Rl = Rp @ self.ETt[idx] @ Rj
            # a prismatic link's origin slides by q a (joint frame) from r_T
            slide = torch.where(pr[:, None], qi[:, None] * self.ax[idx], torch.zeros_like(self.ax[idx]))
            r = self.rT[idx] + (self.ETt[idx] @ slide[..., None])[..., 0]
            pl = pp + (Rp @ r[..., None])[..., 0]
            if len(free):
                rows_R, rows_p = list(Rl.unbind(0)), list(pl.unbind(0))
                for k in free:
                    qo = int(self.qidx_np[int(idx[k])])
                    rows_R[k] = _quat_R(q[qo + 3:qo + 7])
                    rows_p[k] = q[qo:qo + 3]
                Rl, pl = torch.stack(rows_R), torch.stack(rows_p)
            Rw = Rw.index_copy(0, idx, Rl)
            pw = pw.index_copy(0, idx, pl)
        t = self.target
        return pw[t] + (Rw[t] @ self.pts[..., None])[..., 0]
