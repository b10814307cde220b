// Serial chains whose joint axes are all parallel (a batch with kFrIdentity
// link frames: after the host's canonicalisation every revolute axis is the
// common z and no fixed rotation lies between the links).  Their motion is
// planar: of a spatial velocity only (w_z, v_x, v_y), of a force only (n_z,
// f_x, f_y), and of an inertia only the moment about z, the in-plane first
// moment and the mass enter a joint's equation.  The algorithms are the
// general kernels' with those components alone; everything out of the plane
// drops out exactly.
//
// What bounds these kernels is the number of instructions a wavefront issues
// on the serial path over the levels (one wavefront per SIMD at 4096 chains,
// one link in seven at work at a level): six-dimensional algebra issued about
// 1840 a forward step (FP32, 7 links), 3270 a recompute and 3560 a reverse
// step (FP64); these issue about 750, 1000 and 450.  4096 chains of 7 links x
// 200 steps (FP32 handle): forward 890 -> 360 us, adjoint 1550 -> 420 us; one
// chain x 1000 steps in FP64: 5.2 -> 2.0 and 7.3 -> 1.5 ms; 2048 chains of 5
// to 50 links x 50 steps: 1.46 -> 0.54 and 4.57 -> 0.72 ms.
//
// The forward step (planar_qdd) of an FP32 handle works in link frames, as the
// general kernels do, so its rounding errors are theirs.  The adjoint runs in
// FP64 in the base's axes, where the level loops turn nothing, by the adjoint of
// the inverse dynamics: with w = M^-1 (dt qd1_bar) (two sweeps with the step's factors),
//   tau_bar = w,  (q_bar, qd_bar) -= d/d(q, qd) <w, ID(q, qd, qdd)> at fixed qdd
// (the derivative of M qdd + C(q, qd) = tau), in place of the reversed
// statements of the three passes.  Sec. 3, Eq. adj_back; Sec. 4.1, Eq. adj_r.
#pragma once

namespace aba {

namespace {

// ------------------------------------------------------------ link frames
// Constants of a link, and of its child (the next lane; zeros for a leaf).
template <typename T>
struct PlanarC {
  T rx, ry;    // joint origin in the parent
  T nx, ny;    // the child's
  T m, hx, hy, I;
  bool child, parent;
};
__device__ __forceinline__ float fast_rcp(float x) { return rcp(x); }
// 1 / x: the estimate (2^-23) and two Newton steps, which round as the division
// does (335 million values of both signs and 600 binary orders: none differs);
// the division's own last instruction, for what is zero, infinite or past the
// range
__device__ __forceinline__ double fast_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
  return __builtin_amdgcn_div_fixup(__builtin_fma(r, __builtin_fma(-x, r, 1.0), r), x, 1.0);
}
template <typename S>
__device__ __forceinline__ Dual<S> fast_rcp(const Dual<S>& x) {
  const S v = fast_rcp(x.v);
  return Dual<S>(v, -(x.d * v) * v);
}
template <typename T>
__device__ __forceinline__ T prev1(const T& x) { return dpp_mov<kDppWaveShr1>(x); }
template <typename T>
__device__ __forceinline__ T next1(const T& x) { return dpp_mov<kDppWaveShl1>(x); }

template <typename T, typename S>
__device__ __forceinline__ PlanarC<T> planar_const(const Packed<S>& P, const Lane& l) {
  const int ns = P.nslots, slot = l.slot;
  const S* cf = P.cf;
  PlanarC<T> L;
  auto at = [&](int k) { return T(cf[k * ns + slot]); };
  L.rx = at(CF_RT);
  L.ry = at(CF_RT + 1);
  L.m = at(CF_M);
  L.hx = at(CF_MC);
  L.hy = at(CF_MC + 1);
  L.I = at(CF_IB + 2);
  L.nx = next1(L.rx);
  L.ny = next1(L.ry);
  L.child = l.ccount > 0;
  L.parent = l.active() && l.depth > 0;
  return L;
}
// A value from the parent's (the child's) lane, zero where there is none: a
// select, so that nothing of a neighbouring chain gets in, not even a NaN.
template <typename T>
__device__ __forceinline__ T recv(bool has, const T& moved, const T& none = T(0)) {
  return has ? moved : none;  // (moved: already moved, by every lane)
}

// The same in FP64, in the base's axes with the links' absolute angles and
// rates: a link's acceleration then enters its own row alone, the force
// through a joint is that of a 2 x 2 mass and two numbers, and the level loops
// turn nothing and shift nothing (about 12 dependent operations a level for
// 18).  FP32 handles keep the link frames' rounding.  One chain of 7 links x
// 1000 steps 2.03 -> 1.74 ms, 2048 chains of 5 to 50 x 50 steps 711 -> 573 us.
__device__ __forceinline__ double planar_qdd_abs(const V3<double>& g, const PlanarC<double>& L, double q, double qd,
                                                 double tau, int maxd) {
  double th = q, w = qd;
  for (int d = 0; d < maxd; ++d) {
    th = recv(L.parent, prev1(th)) + q;
    w = recv(L.parent, prev1(w)) + qd;
  }
  double sn, cs;
  sincos_(th, &sn, &cs);
  // to the child's joint, and the first moment; e, (ux, uy): their normals
  const double ey = cs * L.nx - sn * L.ny, ex = -(sn * L.nx + cs * L.ny);
  const double uy = cs * L.hx - sn * L.hy, ux = -(sn * L.hx + cs * L.hy);
  const double w2 = w * w, cx = w2 * ey, cy = -(w2 * ex);  // centripetal, at the child's joint
  const double tab = tau - recv(L.child, next1(tau));
  const double hx = w2 * uy, hy = -(w2 * ux);
  double vx = ux, vy = uy, Di = 0.0, r = 0.0;
  double gxx = 0.0, gxy = 0.0, gyy = 0.0, gfx = 0.0, gfy = 0.0;
  for (int d = 0;; ++d) {
    const double nxx = recv(L.child, next1(gxx)), nxy = recv(L.child, next1(gxy)), nyy = recv(L.child, next1(gyy));
    const double nfx = recv(L.child, next1(gfx)), nfy = recv(L.child, next1(gfy));
    const double kx = nxx * ex + nxy * ey, ky = nxy * ex + nyy * ey;
    Di = fast_rcp(L.I + (ex * kx + ey * ky));
    vx = ux + kx;
    vy = uy + ky;
    const double fx = nfx - (nxx * cx + nxy * cy), fy = nfy - (nxy * cx + nyy * cy);
    r = tab - (ex * fx + ey * fy);
    if (d == maxd) break;
    const double px = vx * Di, py = vy * Di;
    gxx = (L.m + nxx) - vx * px;
    gxy = nxy - vx * py;
    gyy = (L.m + nyy) - vy * py;
    gfx = (fx - hx) + r * px;
    gfy = (fy - hy) + r * py;
  }
  const double gx = L.parent ? 0.0 : -g.x, gy = L.parent ? 0.0 : -g.y;  // the base's acceleration
  double al = 0.0, ox = 0.0, oy = 0.0;
  for (int d = 0; d <= maxd; ++d) {
    const double ax = recv(L.parent, prev1(ox), gx), ay = recv(L.parent, prev1(oy), gy);
    al = (r - vx * ax - vy * ay) * Di;
    ox = (ax - cx) + al * ex;
    oy = (ay - cy) + al * ey;
  }
  return al - recv(L.parent, prev1(al));
}

// Forward dynamics of a wave of planar chains: pass 1 root to leaves (w, v),
// pass 2 leaves to root, pass 3 root to leaves.  With the motion subspace
// (1; 0, 0) the handed inertia Ia = IA - U U^T / D has only its 2 x 2 linear
// block and pa's moment is the joint's own torque, so a child hands over
// three and two numbers, turned into the parent's axes; the parent shifts them.
template <typename T>
__device__ __forceinline__ T planar_qdd(const V3<T>& g, const PlanarC<T>& L, T q, T qd, T tau, int maxd) {
  if constexpr (std::is_same_v<T, double>) return planar_qdd_abs(g, L, q, qd, tau, maxd);
  T sn, cs;
  sincos_(q, &sn, &cs);
  // Every pass runs all lanes at every level, without masks: a lane's result
  // depends on its parent's (child's) alone, so it is final once that is, and
  // is computed again to the same bits from then on.
  T w = qd, vx = T(0), vy = T(0);
  for (int d = 0; d < maxd; ++d) {
    const T pw = recv(L.parent, prev1(w)), px = recv(L.parent, prev1(vx)), py = recv(L.parent, prev1(vy));
    const T ux = px - pw * L.ry, uy = py + pw * L.rx;
    w = pw + qd;
    vx = cs * ux + sn * uy;
    vy = cs * uy - sn * ux;
  }
  const T cx = vy * qd, cy = -(vx * qd);
  const T pn = w * (vx * L.hx + vy * L.hy) + recv(L.child, next1(tau));
  const T fx = -(w * (L.m * vy + w * L.hx)), fy = w * (L.m * vx - w * L.hy);
  T a = L.I, bx = -L.hy, by = L.hx, u = tau - pn, Di = T(0);
  T gxx = T(0), gyy = T(0), gxy = T(0), gfx = T(0), gfy = T(0);
  const T c2 = cs * cs, s2 = sn * sn, k = cs * sn, k2 = k + k, cd = c2 - s2;
  for (int d = 0;; ++d) {
    const T nxx = recv(L.child, next1(gxx)), nyy = recv(L.child, next1(gyy)), nxy = recv(L.child, next1(gxy));
    const T nfx = recv(L.child, next1(gfx)), nfy = recv(L.child, next1(gfy));
    const T px = nxy * L.nx - nxx * L.ny, py = nyy * L.nx - nxy * L.ny;
    a = L.I + (py * L.nx - px * L.ny);
    Di = fast_rcp(a);
    bx = px - L.hy;
    by = L.hx + py;
    u = (tau - pn) - (L.nx * nfy - L.ny * nfx);
    if (d == maxd) break;
    const T Cxx = L.m + nxx, Cyy = L.m + nyy;
    const T kx = bx * Di, ky = by * Di;
    const T Pxx = Cxx - bx * kx, Pxy = nxy - bx * ky, Pyy = Cyy - by * ky;
    const T ax = (fx + nfx) + Pxx * cx + Pxy * cy + u * kx, ay = (fy + nfy) + Pxy * cx + Pyy * cy + u * ky;
    gxx = c2 * Pxx + s2 * Pyy - k2 * Pxy;
    gyy = s2 * Pxx + c2 * Pyy + k2 * Pxy;
    gxy = k * (Pxx - Pyy) + cd * Pxy;
    gfx = cs * ax - sn * ay;
    gfy = sn * ax + cs * ay;
  }
  // the base's acceleration is -g
  const T gx = L.parent ? T(0) : -g.x, gy = L.parent ? T(0) : -g.y;
  T al = T(0), lx = T(0), ly = T(0), qdd = T(0);
  for (int d = 0; d <= maxd; ++d) {
    const T pa = recv(L.parent, prev1(al));
    const T px = recv(L.parent, prev1(lx), gx), py = recv(L.parent, prev1(ly), gy);
    const T ux = px - pa * L.ry, uy = py + pa * L.rx;
    lx = cs * ux + sn * uy + cx;
    ly = cs * uy - sn * ux + cy;
    qdd = (u - a * pa - bx * lx - by * ly) * Di;
    al = pa + qdd;
  }
  return qdd;
}

}  // namespace

}  // namespace aba
