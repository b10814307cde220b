"""The contact kernels (csrc/contact.hip, with every lane of a wavefront) on the
CPU, against the FP64 oracle: an unfilled last wavefront, trees with fewer and
with as many links as lanes, both gradient kernels; nothing written outside
the outputs or the launch's LDS."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import contact_cases as CC
import oracle as O
from helpers import rel
from paper_2109_07719_amd import synth
from paper_2109_07719_amd.contact import _Model, _Tiling, pack_params
from test_host_contact import G, _world_point

HERE = os.path.dirname(os.path.abspath(__file__))
DT, NITER, T, GUARD = 1e-3, 10, 3, 64


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("lanes") / "libcontactlanes.so")
    src = os.path.join(HERE, "hostemu", "lanes")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-w", "-I", src, "-o", so,
                           os.path.join(src, "contact_lanes.cpp")])
    L = ctypes.CDLL(so)
    P, I, D = ctypes.c_void_p, ctypes.c_int, ctypes.c_double
    L.sim_contact_rollout.argtypes = [P, I, I, P, P, P, P, D, I, P, P, P, P, P]
    L.sim_contact_rollout_grad.argtypes = [P, I, I, P, P, P, D, I, P, P, P, P, P, P, P]
    L.lanes_overruns.restype = ctypes.c_long
    L.lanes_log.restype = ctypes.c_char_p
    return L


def _p(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def guarded(shape, dtype):
    """An array between two bands of GUARD elements, all of it bytes 0xa5."""
    n = int(np.prod(shape))
    whole = np.frombuffer(bytearray(b"\xa5" * ((n + 2 * GUARD) * np.dtype(dtype).itemsize)), dtype)
    return whole, whole[GUARD:GUARD + n].reshape(shape)


def scene(name):
    if name == "quadruped":
        s, q0, qd0, tau, links, centers, radii = CC.landing_quadruped(3100, T, drop=-1e-3)
    elif name == "chain":
        s, q0, qd0, tau, links, centers, radii = CC.resting_chain(T)
    else:
        s, q0, qd0, tau = synth.tree_system(3, T, nmin=16, nmax=16, random_frames=True, max_depth=16)
        links, radii = np.array([5, 9, 15, 15], np.int32), np.full(4, 0.05)
        centers = np.random.default_rng(3).normal(size=(4, 3)) * 0.1
        s = CC.lower_to_ground(s, q0, links, centers, radii, _world_point, 3e-3)
    return s, q0, qd0, tau, links, centers, radii


@pytest.mark.parametrize("fp64", [True, False], ids=["fp64", "fp32"])
@pytest.mark.parametrize("cus", [0, 256], ids=["a-wavefront", "two-wavefronts"])
@pytest.mark.parametrize("B", [1, 6])
@pytest.mark.parametrize("name", ["quadruped", "chain", "16-link tree"])
def test_kernels_match_the_oracle(lib, name, B, cus, fp64):
    s, q0, qd0, tau, links, centers, radii = scene(name)
    rng = np.random.default_rng(B)
    dtype = np.float64 if fp64 else np.float32
    mu, beta = 0.7, 0.1
    keep = [np.ascontiguousarray(x, np.int32) for x in (s.parent, s.jtype, links)]
    tiling = _Tiling(8, 16, 1)
    m = _Model(s.n, keep[0].ctypes.data, keep[1].ctypes.data, len(links), keep[2].ctypes.data, mu, beta, NITER,
               (ctypes.c_double * 3)(*G), None, ctypes.addressof(tiling))
    rep = lambda x: np.repeat(np.asarray(x, np.float64)[..., None], B, -1).astype(dtype)
    P, q, qd = (np.ascontiguousarray(rep(x)) for x in (pack_params(s, centers, radii), q0, qd0))
    u = np.ascontiguousarray(rep(tau) * (1 + 0.1 * rng.normal(size=(T, 1, B)))).astype(dtype)
    a, b = (rng.normal(size=(n, B)).astype(dtype) for n in (s.nq, s.nv))
    outs = [guarded(x, dtype) for x in ((T + 1, s.nq + s.nv, B), (s.nq, B), (s.nv, B), (s.nq, B), (s.nv, B),
                                        (T, s.nu, B), (B,))] + [guarded((T, B), np.int32)]
    tr, qT, qdT, gq, gqd, gu, gmu, nc = (o[1] for o in outs)
    lib.lanes_set_compute_units(cus)
    lib.lanes_overruns(), lib.lanes_log()
    code = int(fp64)
    assert lib.sim_contact_rollout(ctypes.byref(m), code, B, _p(P), _p(q), _p(qd), _p(u), DT, T, _p(tr), _p(qT),
                                   _p(qdT), _p(nc), None) == 0
    assert lib.sim_contact_rollout_grad(ctypes.byref(m), code, B, _p(P), _p(tr), _p(u), DT, T, _p(a), _p(b), _p(gq),
                                        _p(gqd), _p(gu), _p(gmu), None) == 0
    log = lib.lanes_log().decode()
    assert ("k_contact_adj_pair" in log) == (cus > 0), log
    assert lib.lanes_overruns() == 0
    for whole, _ in outs:
        w = whole.view(np.uint8).reshape(-1)
        g = GUARD * whole.itemsize
        assert (w[:g] == 0xa5).all() and (w[-g:] == 0xa5).all()
    def along(g):
        """g along the unit sphere of a free root's quaternion (across it, a
        step reads contact in no one way)."""
        g = g.copy()
        if s.jtype[0] == synth.FREE:
            g[3:7] -= q0[3:7] * (q0[3:7] @ g[3:7])
        return g

    mo = O.Model(s, G)
    C = O.Contacts(links, centers, radii, mu=mu, beta=beta, niter=NITER)
    assert nc.max() > 0
    for i in range(B) if fp64 else ():
        _, _, nco, tro = O.rollout_contact(mo, C, q[:, i], qd[:, i], u[:, :, i], DT, traj=True)
        assert np.array_equal(nco, nc[:, i])
        assert rel(tr[1:, :, i], tro, 1e-12) < 1e-10 and np.array_equal(tr[-1, :, i], np.r_[qT[:, i], qdT[:, i]])
        ref = O.rollout_contact_grad(mo, C, q[:, i], qd[:, i], u[:, :, i], DT, a[:, i], b[:, i], mu_grad=True)
        scale = max(np.abs(r).max() for r in ref[:3] if r.size)
        for x, r in zip((along(gq[:, i]), gqd[:, i], gu[:, :, i], gmu[i]), (along(ref[0]),) + ref[1:]):
            assert rel(x, np.asarray(r), 1e-6 * scale) < 1e-8
    assert all(np.isfinite(o[1]).all() for o in outs[:-1])
