// The adjoint of planar chains in the base's axes (planar.h: what planar
// means here, and the adjoint's formulas).  Included by abadj_device.h after
// the general backward kernels.
//
// A link's quantities are taken about its own joint's origin, where the motion
// subspace is (1; 0, 0): the inertia handed to the parent then has only its 2 x
// 2 linear block, the moment handed is the joint's own torque, and the parent
// shifts both by the step to its child.  About the base's origin an inertia
// holds the squared distance, and a joint's small part is what is left of it.
// Error of tau_bar, one step of 20 links in FP64, link frames / the base's
// origin / own origins: 3.0e-16 / 4.7e-15 / 2.9e-16, mounted 10 m off it 3.0e-16
// / 3.0e-13 / 2.9e-16.
// It is also the shorter: a level hands on five numbers instead of nine (4096
// chains of 7 links x 200 steps, forward and adjoint 720 -> 708 us, 2048 chains
// of 5 to 50 x 50 1367 -> 1282).
#pragma once

#include "planar.h"

namespace aba {

namespace {

struct P3 {  // motion (w; v_x, v_y) or force (n; f_x, f_y)
  double w, x, y;
};
__device__ __forceinline__ P3 operator+(const P3& a, const P3& b) { return {a.w + b.w, a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ P3 operator-(const P3& a, const P3& b) { return {a.w - b.w, a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ P3 operator*(double s, const P3& a) { return {s * a.w, s * a.x, s * a.y}; }
__device__ __forceinline__ double dot(const P3& a, const P3& b) { return a.w * b.w + a.x * b.x + a.y * b.y; }
// crm, crf, crm^T of spatial.h
__device__ __forceinline__ P3 crm(const P3& a, const P3& b) {
  return {0.0, b.w * a.y - a.w * b.y, a.w * b.x - b.w * a.x};
}
__device__ __forceinline__ P3 crf(const P3& a, const P3& f) { return {a.x * f.y - a.y * f.x, -(a.w * f.y), a.w * f.x}; }
__device__ __forceinline__ P3 crmT(const P3& a, const P3& x) {
  return {x.x * a.y - x.y * a.x, a.w * x.y, -(a.w * x.x)};
}
__device__ __forceinline__ P3 prev3(bool has, const P3& a) {
  return {recv(has, prev1(a.w)), recv(has, prev1(a.x)), recv(has, prev1(a.y))};
}
__device__ __forceinline__ P3 next3(bool has, const P3& a) {
  return {recv(has, next1(a.w)), recv(has, next1(a.x)), recv(has, next1(a.y))};
}

struct PlanarLane {
  int dep, below;  // level (-1: idle lane); links below it in its chain
  int maxd;
  bool parent, child;
  double rx, ry, m, hx, hy, I, gx, gy;
};
template <typename S>
__device__ __forceinline__ PlanarLane planar_lane(const Packed<S>& P, const Lane& l, int maxd) {
  const PlanarC<double> L = planar_const<double>(P, l);
  PlanarLane p;
  p.dep = l.active() ? l.depth : -1;
  p.maxd = maxd;
  p.parent = L.parent;
  p.child = L.child;
  p.rx = L.rx;
  p.ry = L.ry;
  p.m = L.m;
  p.hx = L.hx;
  p.hy = L.hy;
  p.I = L.I;
  p.gx = double(P.g[0]);
  p.gy = double(P.g[1]);
  p.below = 0;
  for (int d = maxd; d > 0; --d) {
    const int n = __builtin_amdgcn_update_dpp(0, p.below, kDppWaveShl1, 0xf, 0xf, true);
    if (l.ccount > 0 && p.dep == d - 1) p.below = n + 1;
  }
  return p;
}

// Sums over a link's ancestors and itself, and over its descendants and
// itself.  Short chains step from level to level by DPP; from 16 levels up
// the sums go over 1, 2, 4, ... lanes through ds_bpermute (six rounds for 50
// links in place of 49 steps; below that the rounds' LDS latency costs more).
constexpr int kScanLevels = 16;
template <int N>
__device__ __forceinline__ void sum_down(const PlanarLane& p, double (&v)[N]) {
  if (p.maxd < kScanLevels) {
    double own[N];
#pragma unroll
    for (int k = 0; k < N; ++k) own[k] = v[k];
    for (int d = 0; d < p.maxd; ++d) {
#pragma unroll
      for (int k = 0; k < N; ++k) v[k] = recv(p.parent, prev1(v[k])) + own[k];
    }
  } else {
    for (int s = 1; s <= p.maxd; s <<= 1) {
      double t[N];
#pragma unroll
      for (int k = 0; k < N; ++k) t[k] = __shfl_up(v[k], s);
      if (p.dep >= s) {
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = t[k] + v[k];
      }
    }
  }
}
// Two forces (v[0..2], v[3..5]: moment, x, y), each about its link's own
// origin; (cx, cy): the step to the child's.
__device__ __forceinline__ void sum_up(const PlanarLane& p, double cx, double cy, double (&v)[6]) {
  if (p.maxd < kScanLevels) {
    double own[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) own[k] = v[k];
    for (int d = 0; d < p.maxd; ++d) {
      double t[6];
#pragma unroll
      for (int k = 0; k < 6; ++k) t[k] = recv(p.child, next1(v[k]));
#pragma unroll
      for (int k = 0; k < 6; k += 3) {
        v[k] = own[k] + (t[k] + (cx * t[k + 2] - cy * t[k + 1]));
        v[k + 1] = own[k + 1] + t[k + 1];
        v[k + 2] = own[k + 2] + t[k + 2];
      }
    }
  } else {
    for (int s = 1; s <= p.maxd; s <<= 1) {  // (cx, cy): the step over s links
      double t[6];
#pragma unroll
      for (int k = 0; k < 6; ++k) t[k] = __shfl_down(v[k], s);
      const double tx = __shfl_down(cx, s), ty = __shfl_down(cy, s);
      if (p.below >= s) {
#pragma unroll
        for (int k = 0; k < 6; k += 3) {
          v[k] = v[k] + (t[k] + (cx * t[k + 2] - cy * t[k + 1]));
          v[k + 1] = v[k + 1] + t[k + 1];
          v[k + 2] = v[k + 2] + t[k + 2];
        }
        cx += tx;
        cy += ty;
      }
    }
  }
}

// What the reverse of a step reads of it.
struct PlanarTape {
  double dx, dy;         // the parent's origin to the link's (a root: zero)
  P3 U;
  double Di;
  P3 V;
  double hx, hy;         // first moment
  P3 Ap, F;              // the parent's acceleration; the force through the joint
  double qd;
};
constexpr int kPlanarTape = 18;

// The step's factors, velocities, accelerations and joint forces at (q, qd)
// under tau.
__device__ __forceinline__ PlanarTape planar_recompute(const PlanarLane& p, double q, double qd, double tau) {
  PlanarTape o;
  o.qd = qd;
  double th[1] = {q};
  sum_down(p, th);
  double sn, cs;
  sincos(th[0], &sn, &cs);
  const double ps = prev1(sn), pc = prev1(cs);
  o.dx = p.parent ? pc * p.rx - ps * p.ry : 0.0;
  o.dy = p.parent ? ps * p.rx + pc * p.ry : 0.0;
  double w[1] = {qd};
  sum_down(p, w);
  const double wp = recv(p.parent, prev1(w[0]));
  double v[2] = {-(wp * o.dy), wp * o.dx};
  sum_down(p, v);
  o.V = {w[0], v[0], v[1]};
  const P3 cb = crm(o.V, P3{qd, 0.0, 0.0});
  double ab[2] = {cb.x, cb.y};
  sum_down(p, ab);  // (no angular part: nothing to shift)
  const P3 A0 = {0.0, ab[0] - p.gx, ab[1] - p.gy};
  o.hx = cs * p.hx - sn * p.hy;
  o.hy = sn * p.hx + cs * p.hy;
  const P3 h = {p.I * o.V.w + o.hx * o.V.y - o.hy * o.V.x, p.m * o.V.x - o.V.w * o.hy, p.m * o.V.y + o.V.w * o.hx};
  P3 F = P3{o.hx * A0.y - o.hy * A0.x, p.m * A0.x, p.m * A0.y} + crf(o.V, h);
  F.w = F.w + recv(p.child, next1(tau));
  const double cx = recv(p.child, next1(o.dx)), cy = recv(p.child, next1(o.dy));
  double Cxx, Cxy, Cyy, Fx, Fy, u;
  double gxx = 0, gxy = 0, gyy = 0, gfx = 0, gfy = 0;
  for (int d = 0;; ++d) {
    const double nxx = recv(p.child, next1(gxx)), nxy = recv(p.child, next1(gxy)), nyy = recv(p.child, next1(gyy));
    const double nfx = recv(p.child, next1(gfx)), nfy = recv(p.child, next1(gfy));
    const double kx = nxy * cx - nxx * cy, ky = nyy * cx - nxy * cy;
    o.U = {p.I + (ky * cx - kx * cy), kx - o.hy, o.hx + ky};
    o.Di = fast_rcp(o.U.w);
    Cxx = p.m + nxx;
    Cxy = nxy;
    Cyy = p.m + nyy;
    Fx = F.x + nfx;
    Fy = F.y + nfy;
    u = tau - (F.w + (cx * nfy - cy * nfx));
    if (d == p.maxd) break;
    const double bx = o.U.x * o.Di, by = o.U.y * o.Di;
    gxx = Cxx - o.U.x * bx;
    gxy = Cxy - o.U.x * by;
    gyy = Cyy - o.U.y * by;
    gfx = Fx + u * bx;
    gfy = Fy + u * by;
  }
  P3 ap = {0, 0, 0}, ac = {u * o.Di, 0, 0};
  for (int d = 0; d < p.maxd; ++d) {
    const P3 t = prev3(p.parent, ac);
    ap = {t.w, t.x - t.w * o.dy, t.y + t.w * o.dx};
    ac = {ap.w + (u - dot(o.U, ap)) * o.Di, ap.x, ap.y};
  }
  // the joint's force is IA a + pA, its moment the torque; the parent's
  // acceleration with its bias
  o.F = {tau, o.U.x * ac.w + Cxx * ac.x + Cxy * ac.y + Fx, o.U.y * ac.w + Cxy * ac.x + Cyy * ac.y + Fy};
  o.Ap = ap + A0 - cb;
  return o;
}

// The adjoint of the step: (xq, xqd) in, the adjoint of (q1, qd1), and out,
// that of (q, qd); returns tau_bar.
__device__ __forceinline__ double planar_reverse(const PlanarLane& p, const PlanarTape& o, double dt, double& xq,
                                                 double& xqd) {
  const double tot = xqd + dt * xq;
  const double r0 = dt * tot, rc = recv(p.child, next1(r0));
  const double cx = recv(p.child, next1(o.dx)), cy = recv(p.child, next1(o.dy));
  double r = r0, px = 0, py = 0;  // (r0; px, py): the force handed on
  for (int d = 0;; ++d) {
    const double nx = recv(p.child, next1(px)), ny = recv(p.child, next1(py));
    r = r0 - (rc + (cx * ny - cy * nx));
    if (d == p.maxd) break;
    const double k = r * o.Di;
    px = nx + k * o.U.x;
    py = ny + k * o.U.y;
  }
  double w = r * o.Di;
  P3 B = {w, 0, 0}, Bp = {0, 0, 0};
  for (int d = 0; d < p.maxd; ++d) {
    const P3 t = prev3(p.parent, B);
    Bp = {t.w, t.x - t.w * o.dy, t.y + t.w * o.dx};
    w = (r - dot(o.U, Bp)) * o.Di;
    B = {Bp.w + w, Bp.x, Bp.y};
  }
  auto mul = [&](const P3& a) {
    return P3{p.I * a.w + o.hx * a.y - o.hy * a.x, p.m * a.x - a.w * o.hy, p.m * a.y + a.w * o.hx};
  };
  // <w, ID> = sum_i B_i . (I A + V x* I V): per link its share of A's adjoint,
  // I B, and of V's; the bias accelerations V_l x S_l qd_l between the root
  // and link i sum to V_i in the second
  const P3 IB = mul(B), e = crmT(B, mul(o.V)) - mul(crm(o.V, B)) - crmT(o.V, IB);
  double s[6] = {IB.w, IB.x, IB.y, e.w, e.x, e.y};
  sum_up(p, cx, cy, s);
  const P3 G = {s[0], s[1], s[2]};
  const P3 Vp = {o.V.w - o.qd, o.V.x, o.V.y};
  const P3 vb = P3{s[3], s[4], s[5]} + crmT(Vp, G);
  // the subtree turns with q: what enters it from the parent turns back
  xq = xq + (crf(Bp, o.F).w + crf(o.Ap, G).w + crf(Vp, vb).w);
  xqd = tot - (crmT(o.V, G).w + vb.w);
  return w;
}

__device__ __forceinline__ void put_planar(const PlanarTape& o, double* b, int lane) {
  const double v[kPlanarTape] = {o.dx,   o.dy,   o.U.w,  o.U.x, o.U.y, o.Di,  o.V.w, o.V.x, o.V.y,
                                 o.hx,   o.hy,   o.Ap.w, o.Ap.x, o.Ap.y, o.F.w, o.F.x, o.F.y, o.qd};
#pragma unroll
  for (int k = 0; k < kPlanarTape; ++k) b[k * kWave + lane] = v[k];
}
__device__ __forceinline__ PlanarTape get_planar(const double* b, int lane) {
  auto at = [&](int k) { return b[k * kWave + lane]; };
  PlanarTape o;
  o.dx = at(0);
  o.dy = at(1);
  o.U = {at(2), at(3), at(4)};
  o.Di = at(5);
  o.V = {at(6), at(7), at(8)};
  o.hx = at(9);
  o.hy = at(10);
  o.Ap = {at(11), at(12), at(13)};
  o.F = {at(14), at(15), at(16)};
  o.qd = at(17);
  return o;
}

// Writes a step's tau_bar and adds the trajectory's seed of x^t.
template <typename S>
__device__ __forceinline__ void planar_outputs(const BwdArgs<S>& A, const Lane& l, int t, double taub, double& xq,
                                               double& xqd, int& nonfin) {
  if (!l.active()) return;
  const S out = S(taub);
  A.gtau[(size_t)t * A.P.nu + l.uidx] = out;
  nonfin += nonfinite(out);
  if (A.gtraj != nullptr && t >= 1) {
    const S* row = A.gtraj + (size_t)(t - 1) * (A.P.nq + A.P.nv);
    xq += double(row[l.qidx]);
    xqd += double(row[A.P.nq + l.vidx]);
  }
}

// The backward rollout of planar chains, one wavefront: K == 1 reloads every
// checkpoint, K > 1 replays each segment into the scratch buffer, K < 0 runs
// the binomial schedule (as k_backward).
template <typename S>
__global__ __launch_bounds__(kWave * kMaxWavesPerBlock) void k_backward_planar(BwdArgs<S> A) {
  const int wb = wave_batch();
  const Lane l = load_lane(A.P, wb);
  const int maxd = wave_maxd(A.P, wb);
  const int ns = A.P.nslots, nu = A.P.nu;
  const size_t RW = state_record(ns, A.P.nfree);
  const bool act = l.active();
  const PlanarLane p = planar_lane(A.P, l, maxd);
  const PlanarC<S> L = planar_const<S>(A.P, l);
  const V3<S> g = gravity(A.P);
  const double dt = double(A.dt);
  int nonfin = 0;
  const State<double, false> x0 = seed_state<S, double, false>(A, l);
  double xq = x0.q[0], xqd = x0.qd[0];
  auto reverse = [&](S q, S qd, S tau, int t) {
    const PlanarTape o = planar_recompute(p, double(q), double(qd), double(tau));
    const double taub = planar_reverse(p, o, dt, xq, xqd);
    planar_outputs(A, l, t, taub, xq, xqd, nonfin);
  };
  auto ctl = [&](int t) { return act ? A.tau[(size_t)t * nu + l.uidx] : S(0); };
  auto get = [&](const S* rec, S& q, S& qd) {
    q = act ? rec[l.slot] : S(0);
    qd = act ? rec[ns + l.slot] : S(0);
  };
  auto put = [&](S* rec, S q, S qd) {
    if (act) {
      rec[l.slot] = q;
      rec[ns + l.slot] = qd;
    }
  };
  auto advance = [&](S& q, S& qd, S tau) {
    const S qdd = planar_qdd<S>(g, L, q, qd, tau, maxd);
    if (act) integrate_joint(q, qd, qdd, A.dt);
  };
  if (A.K < 0) {
    S q = S(0), qd = S(0);
    int tc = 0;
    for (int i = 0; i < A.nsched; ++i) {
      const int op = A.sched[2 * i], arg = A.sched[2 * i + 1];
      const int what = op & 7, slot = op >> 3;
      if (what == SCH_RESTORE) {
        get(A.ck + (size_t)slot * RW, q, qd);
        tc = arg;
      } else if (what == SCH_ADVANCE) {
        for (int j = 0; j < arg; ++j, ++tc) advance(q, qd, ctl(tc));
      } else if (what == SCH_TAKESHOT) {
        put(A.ck + (size_t)slot * RW, q, qd);
      } else {
        reverse(q, qd, ctl(arg), arg);
      }
    }
  } else {
    const int seg = A.K == 1 ? max(A.T, 1) : A.K;  // K == 1: every state is stored
    const int ncp = (A.T + seg - 1) / seg;
    for (int s = ncp - 1; s >= 0; --s) {
      const int t0 = s * seg, t1 = min(t0 + seg, A.T);
      const S* base = A.ck + (size_t)s * RW;  // states of the segment's steps
      if (A.K > 1) {
        S q, qd;
        get(base, q, qd);
        put(A.scratch, q, qd);
        for (int j = 1; j < t1 - t0; ++j) {
          advance(q, qd, ctl(t0 + j - 1));
          put(A.scratch + (size_t)j * RW, q, qd);
        }
        base = A.scratch;
      }
      // the next state is fetched while this one is reversed
      S nq, nqd, nt = ctl(t1 - 1);
      get(base + (size_t)(t1 - 1 - t0) * RW, nq, nqd);
      for (int t = t1 - 1; t >= t0; --t) {
        const S q = nq, qd = nqd, tau = nt;
        if (t > t0) {
          get(base + (size_t)(t - 1 - t0) * RW, nq, nqd);
          nt = ctl(t - 1);
        }
        reverse(q, qd, tau, t);
      }
    }
  }
  if (act) {
    const S q = S(xq), qd = S(xqd);
    A.gq0[l.qidx] = q;
    A.gqd0[l.vidx] = qd;
    nonfin += nonfinite(q) + nonfinite(qd);
  }
  report_nonfinite(A.P.status, nonfin);
}

// Pipelined, K == 1: NP wavefronts recompute while one reverses.  The steps'
// recomputes do not depend on one another, so in phase k producer j
// recomputes step k NP + j (counted from the end) into buffer k % 2 while the
// consumer reverses the NP steps of phase k - 1; a workgroup barrier ends
// every phase.
template <int NP>
constexpr size_t planar_lds_per_group() {
  return (size_t)2 * NP * kPlanarTape * kWave * sizeof(double);
}
template <typename S, int NP>
__global__ __launch_bounds__((NP + 1) * kWave * kMaxPairsPerBlock) void k_backward_planar_pipe(BwdArgs<S> A) {
  constexpr int G = (NP + 1) * kWave, TW = kPlanarTape * kWave;
  const int group = threadIdx.x / G, wid = threadIdx.x % G / kWave;
  double* const buf = reinterpret_cast<double*>(abadj_lds + group * planar_lds_per_group<NP>());
  const int wb = blockIdx.x * (blockDim.x / G) + group;
  const Lane l = load_lane(A.P, wb);
  const int maxd = wave_maxd(A.P, wb);
  const int ns = A.P.nslots, nu = A.P.nu, T = A.T;
  const size_t RW = state_record(ns, A.P.nfree);
  const bool act = l.active();
  const PlanarLane p = planar_lane(A.P, l, maxd);
  const int phases = (T + NP - 1) / NP;
  if (wid < NP) {
    S nq = S(0), nqd = S(0), nt = S(0);
    auto fetch = [&](int t) {
      if (t >= 0 && act) {
        const S* rec = A.ck + (size_t)t * RW;
        nq = rec[l.slot];
        nqd = rec[ns + l.slot];
        nt = A.tau[(size_t)t * nu + l.uidx];
      }
    };
    fetch(T - 1 - wid);
    for (int k = 0; k <= phases; ++k) {
      const int t = T - 1 - (k * NP + wid);
      if (k < phases && t >= 0) {
        const double q = double(nq), qd = double(nqd), tau = double(nt);
        fetch(t - NP);
        put_planar(planar_recompute(p, q, qd, tau), buf + ((k & 1) * NP + wid) * TW, l.lane);
      }
      __syncthreads();
    }
  } else {
    const double dt = double(A.dt);
    int nonfin = 0;
    const State<double, false> x0 = seed_state<S, double, false>(A, l);
    double xq = x0.q[0], xqd = x0.qd[0];
    for (int k = 0; k <= phases; ++k) {
      for (int j = 0; j < NP; ++j) {
        const int t = T - 1 - ((k - 1) * NP + j);
        if (k > 0 && t >= 0) {
          const PlanarTape o = get_planar(buf + (((k - 1) & 1) * NP + j) * TW, l.lane);
          const double taub = planar_reverse(p, o, dt, xq, xqd);
          planar_outputs(A, l, t, taub, xq, xqd, nonfin);
        }
      }
      __syncthreads();
    }
    if (act) {
      const S q = S(xq), qd = S(xqd);
      A.gq0[l.qidx] = q;
      A.gqd0[l.vidx] = qd;
      nonfin += nonfinite(q) + nonfinite(qd);
    }
    report_nonfinite(A.P.status, nonfin);
  }
}

}  // namespace

}  // namespace aba
