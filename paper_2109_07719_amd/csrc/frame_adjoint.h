// The FP64 adjoint of trees, free roots, prismatic and ball joints and joint
// limits, in the base frame, by the adjoint of the inverse dynamics: with w =
// M^-1 (dt qd1_bar) (two sweeps with the step's articulated factors),
//   tau_bar = w,  (q_bar, qd_bar) -= d/d(q, qd) <w, ID(q, qd, qdd)> at fixed qdd
// (the derivative of M qdd + C(q, qd) = tau).  Sec. 3, Eq. adj_back; Sec. 4.1,
// Eq. adj_r.  Included by abadj_device.h after the general backward kernels.
//
// What bounds these kernels is the instructions a wavefront issues over the
// levels of a tree, where one lane in six works.  So every spatial quantity is
// in the axes of one frame (a fixed base's; a free root's own, where its motion
// subspace is the identity): the level loops rotate nothing, poses and
// velocities come from ancestor-doubling rounds (log2 of the depth) instead of
// levels, and what the reverse needs beyond the two sweeps is one sum over each
// subtree.  Adjoints of 8192 trees x 50 steps 2.83 -> 1.60 ms, of 1024
// quadrupeds x 200 steps in segments of 10 (replay included) 4.74 -> 2.86 ms.
//
// Where they are taken about is a matter of the handle's type (kOwnOrigin).  An
// FP32 handle's: about the root's joint origin, and nothing is shifted either.
// An inertia there holds the squared distance from it, and a joint's small
// numbers are what is left of that; FP32 outputs do not show it.  An FP64
// handle's: each link's about its own joint's origin, shifted by d, the step
// from the parent's origin to the link's, where they pass from link to link.
// Error of tau_bar, one step of a 20-link tree in FP64, link frames / one
// origin / own origins: 2.5e-16 / 1.8e-15 / 4.0e-16 (a fixed base's own place
// is left out of all three).  8192 trees x 50 steps in an FP32 handle with own
// origins: 1.60 -> 1.90 ms.
//
// A ball joint's three axes turn with its link; its subspace is every
// rotation about the joint's origin o, S = [1; [o]x], and its block form is
// taken about o, where S = [1; 0] (aba_lane.h, "ball joint").  A quaternion off
// the unit sphere scales the joint's transform by |quat|^2 (as the step does):
// the pose takes the rotation alone, and whatever passes through the joint,
// motions down and forces up, is multiplied.
#pragma once

#include "planar_adjoint.h"

namespace aba {

namespace {

constexpr int kJumps = 6;  // doubling rounds for up to 64 levels

template <typename S>
constexpr bool kOwnOrigin = sizeof(S) == sizeof(double);

// The link's constants stay in the handle's type S (FP32 ones widen exactly
// where they are used, at a third of the registers' cost).
template <typename S>
struct FrameLane {
  int lane, par, dep, cf, cc, maxd;
  int base;         // the lane of the system's free root, -1 without one
  int anc[kJumps];  // the lane 1, 2, 4, ... levels up, -1 past the root
  bool act, one, root, ball, prism;
  LinkC<S> L;
  V3<S> g;
};

template <typename S, int FR>
__device__ __forceinline__ FrameLane<S> frame_lane(const Packed<S>& P, const Lane& l, int maxd) {
  FrameLane<S> p;
  p.L = load_linkc<S, FR>(P, l);
  p.lane = l.lane;
  p.par = l.active() ? l.par : -1;
  p.dep = l.active() ? l.depth : -1;
  p.cf = l.cfirst;
  p.cc = l.active() ? l.ccount : 0;
  p.maxd = maxd;
  p.act = l.active();
  p.one = l.onedof() && l.active();
  p.root = l.jtype == 1;
  p.ball = FR == kFrBall && l.ball();
  p.prism = p.L.prism;
  p.g = gravity(P);
  int a = p.par;
#pragma unroll
  for (int r = 0; r < kJumps; ++r) {
    p.anc[r] = a;
    const int up = __shfl(a, a < 0 ? 0 : a);
    a = a < 0 ? -1 : up;
  }
  p.base = p.root ? p.lane : -1;
#pragma unroll
  for (int r = 0; r < kJumps; ++r) {
    const int b = __shfl(p.base, p.anc[r] < 0 ? 0 : p.anc[r]);
    if (p.anc[r] >= 0 && p.base < 0) p.base = b;
  }
  return p;
}

// From one origin to another, d the step from the parent's to the link's: a
// motion goes down it, a force and an inertia up.
__device__ __forceinline__ V6<double> down(const V3<double>& d, const V6<double>& v) {
  return v6<double>(v.a, v.l + cross(v.a, d));
}
__device__ __forceinline__ V6<double> up(const V3<double>& d, const V6<double>& f) {
  return v6<double>(f.a + cross(d, f.l), f.l);
}
__device__ __forceinline__ SySp<double> up(const V3<double>& d, const SySp<double>& M) {
  M3<double> E;
#pragma unroll
  for (int k = 0; k < 9; ++k) E.m[k] = k % 4 == 0 ? 1.0 : 0.0;
  return congruence_XT(E, d, M);
}

// Motions v of the link and its ancestors summed, about the link's origin: by
// doubling rounds through the exchange records (a round: one write and one
// read of every lane).  With own origins a round also carries the step D over
// the links summed so far, with ball joints the scale of their transforms
// (returned: the whole path's).
template <bool BALL, typename S>
__device__ __forceinline__ V6<double> path_sum(const FrameLane<S>& p, V6<double> v, V3<double> D, double& scale,
                                               double* xb) {
#pragma unroll
  for (int r = 0; r < kJumps; ++r) {
    if (1 << r > p.maxd) break;
    put6(xb, 0, p.lane, v);
    if constexpr (kOwnOrigin<S> || BALL) {
      const double t[4] = {D.x, D.y, D.z, scale};
      put_rec(xb, p.lane, 6, t);
    }
    wave_sync();
    if (p.anc[r] >= 0) {
      V6<double> u = get6(xb, 0, p.anc[r]);
      if constexpr (kOwnOrigin<S> || BALL) {
        double t[4];
        get_rec(xb, p.anc[r], 6, t);
        u = down(D, u);
        D = v3<double>(t[0], t[1], t[2]) + D;
        if constexpr (BALL) {
          u = scale * u;
          scale *= t[3];
        }
      }
      v = u + v;
    }
    wave_sync();
  }
  return v;
}

// A step's quantities that its reverse reads.  A free root keeps its 6 x 6
// factor M = L^T D L in ax, U, Di, Ap, F (root_pack), which it does not use.
struct FrameStep {
  V3<double> ax;         // the 1-dof joint's axis
  V3<double> at;         // the joint's origin; with own origins from the parent's (a root: zero)
  V6<double> U, V, Ap, F;
  double Di;
  V3<double> mc;
  Sy3<double> I;
  double q, qd;          // 1-dof joint
  V6<double> abase;      // free root: acceleration; ball: [acceleration, (|quat|^2, 0, 0)]
  // ball joint
  M3<double> R, B;       // pose; the articulated inertia's coupling block about o
  Sy3<double> Ai;        // inverse of its angular block
};

struct RootF {
  double L[15], iv[6];
};
__device__ __forceinline__ void root_pack(FrameStep& o, const RootF& f) {
  const double* L = f.L;
  o.ax = v3<double>(L[0], L[1], L[2]);
  o.U = v6<double>(v3<double>(L[3], L[4], L[5]), v3<double>(L[6], L[7], L[8]));
  o.Di = L[9];
  o.Ap = v6<double>(v3<double>(L[10], L[11], L[12]), v3<double>(L[13], L[14], f.iv[0]));
  o.F = v6<double>(v3<double>(f.iv[1], f.iv[2], f.iv[3]), v3<double>(f.iv[4], f.iv[5], 0.0));
}
__device__ __forceinline__ RootF root_unpack(const FrameStep& o) {
  return {{o.ax.x, o.ax.y, o.ax.z, o.U.a.x, o.U.a.y, o.U.a.z, o.U.l.x, o.U.l.y, o.U.l.z, o.Di, o.Ap.a.x, o.Ap.a.y,
           o.Ap.a.z, o.Ap.l.x, o.Ap.l.y},
          {o.Ap.l.z, o.F.a.x, o.F.a.y, o.F.a.z, o.F.l.x, o.F.l.y}};
}
__device__ __forceinline__ RootF root_factor(const SySp<double>& IA) {
  double M[36];
  sysp_dense(IA, M);
  RootF f;
#pragma unroll
  for (int k = 5; k >= 0; --k) {
    f.iv[k] = fast_rcp(M[7 * k]);
#pragma unroll
    for (int i = 0; i < k; ++i) {
      const double c = M[6 * k + i] * f.iv[k];
      f.L[k * (k - 1) / 2 + i] = c;
#pragma unroll
      for (int j = 0; j <= i; ++j) M[6 * i + j] = fma(-c, M[6 * k + j], M[6 * i + j]);
    }
  }
  return f;
}
__device__ __forceinline__ V6<double> root_solve(const RootF& f, const V6<double>& b) {
  double r[6] = {b.a.x, b.a.y, b.a.z, b.l.x, b.l.y, b.l.z};
#pragma unroll
  for (int e = 5; e >= 0; --e)
#pragma unroll
    for (int i = 0; i < e; ++i) r[i] = fma(-f.L[e * (e - 1) / 2 + i], r[e], r[i]);
#pragma unroll
  for (int e = 0; e < 6; ++e) {
    double v = r[e] * f.iv[e];
#pragma unroll
    for (int i = 0; i < e; ++i) v = fma(-f.L[e * (e - 1) / 2 + i], r[i], v);
    r[e] = v;
  }
  return v6<double>(v3<double>(r[0], r[1], r[2]), v3<double>(r[3], r[4], r[5]));
}

// The rotation nearest to R by one Newton step, R (3 - R^T R) / 2.  The adjoint
// takes R as one (S_k turns with q as S_m x S_k), but widened FP32 frames and
// quaternions are off by 1e-7, and FP64 ones, doubled through a tree, by ten
// roundings.  Error of tau_bar, one step of a 20-link tree, without / with / in
// link frames: FP32 handle 1.0e-7 / 3.6e-8 / 3.8e-8, FP64 2.9e-15 / 4.0e-16 /
// 2.5e-16.
__device__ __forceinline__ M3<double> nearest_rotation(const M3<double>& R) {
  M3<double> G = mul(transpose(R), R);
#pragma unroll
  for (int k = 0; k < 9; ++k) G.m[k] = (k % 4 == 0 ? 1.5 : 0.0) - 0.5 * G.m[k];
  return mul(R, G);
}

// The step from the parent's origin to the link's, and the joint's origin o:
// one of the two is zero (which folds).
template <typename S>
__device__ __forceinline__ V3<double> step_of(const FrameLane<S>&, const FrameStep& o) {
  return kOwnOrigin<S> ? o.at : zero3<double>();
}
template <typename S>
__device__ __forceinline__ V3<double> joint_of(const FrameLane<S>&, const FrameStep& o) {
  return kOwnOrigin<S> ? zero3<double>() : o.at;
}
// the scale of the joint's transform
template <bool BALL, typename S>
__device__ __forceinline__ double scale_of(const FrameLane<S>& p, const FrameStep& o) {
  return BALL && p.ball ? o.abase.l.x : 1.0;
}
// the 1-dof joint's motion subspace
template <typename S>
__device__ __forceinline__ V6<double> subspace(const FrameLane<S>& p, const FrameStep& o) {
  return p.prism ? v6<double>(zero3<double>(), o.ax) : v6<double>(o.ax, cross(joint_of(p, o), o.ax));
}

// half: called half way, by every lane
struct Nothing {
  __device__ void operator()() const {}
};
template <bool FREE, bool BALL, typename S, typename H = Nothing>
__device__ __forceinline__ FrameStep frame_recompute(const FrameLane<S>& p, const State<double, FREE>& st,
                                                     const V3<double>& ctl, double* xb, H&& half = H()) {
  FrameStep o;
  const V3<double> z3 = zero3<double>();
  o.q = st.q[0];
  o.qd = st.qd[0];
  o.abase = zero6<double>();
  // ---- poses by doubling rounds
  M3<double> R;
#pragma unroll
  for (int k = 0; k < 9; ++k) R.m[k] = k % 4 == 0 ? 1.0 : 0.0;
  // the joint's origin from the parent's; own origins: in the link's axes
  V3<double> org = z3;
  const V3<double> grav = widen<double>(p.g);
  V3<double> gb = grav;
  const M3<double> ETt = widen<double>(transpose(p.L.ET));
  const double m = double(p.L.m);
  if (p.one) {
    R = ETt;
    if (!p.prism) {
      double sn, cs;
      sincos(o.q, &sn, &cs);
      // E_T^T times the rotation by q about z
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        R.m[3 * i] = cs * ETt.m[3 * i] + sn * ETt.m[3 * i + 1];
        R.m[3 * i + 1] = cs * ETt.m[3 * i + 1] - sn * ETt.m[3 * i];
      }
    }
    org = widen<double>(p.L.rT);
    if (p.prism) org = axpy(org, o.q, col(ETt, 2));
  }
  if constexpr (BALL) {
    if (p.ball) {
      const Q4<double> q = st_ball_quat(st);
      const double qq = q.x * q.x + q.y * q.y + q.z * q.z + q.w * q.w;
      o.abase.l.x = qq;
      M3<double> Q;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const V3<double> c = (1.0 / qq) * quat_rotate(q, v3<double>(double(j == 0), double(j == 1), double(j == 2)));
        Q.m[j] = c.x;
        Q.m[3 + j] = c.y;
        Q.m[6 + j] = c.z;
      }
      R = mul(ETt, Q);
      org = widen<double>(p.L.rT);
    }
  }
  if (p.par < 0) org = z3;  // where a fixed base stands does not matter
  if constexpr (kOwnOrigin<S>) org = mulT(R, org);
  if constexpr (!kOwnOrigin<S>) R = nearest_rotation(R);
#pragma unroll
  for (int r = 0; r < kJumps; ++r) {
    if (1 << r > p.maxd) break;
    const double t[12] = {R.m[0], R.m[1], R.m[2], R.m[3], R.m[4], R.m[5], R.m[6], R.m[7], R.m[8], org.x, org.y, org.z};
    put_rec(xb, p.lane, 0, t);
    wave_sync();
    if (p.anc[r] >= 0) {
      double u[12];
      get_rec(xb, p.anc[r], 0, u);
      M3<double> Rp;
#pragma unroll
      for (int k = 0; k < 9; ++k) Rp.m[k] = u[k];
      if constexpr (!kOwnOrigin<S>) org = v3<double>(u[9], u[10], u[11]) + mul(Rp, org);
      R = mul(Rp, R);
    }
    wave_sync();
  }
  if constexpr (kOwnOrigin<S>) R = nearest_rotation(R);
  // ---- velocities and bias accelerations (a free root's in the frame that
  // moves with its linear velocity, an exact shift)
  o.ax = col(R, 2);
  if constexpr (kOwnOrigin<S>) o.at = mul(R, org);
  else o.at = org;
  const V3<double> sh = step_of(p, o), oj = joint_of(p, o);
  const double ks = scale_of<BALL>(p, o);
  const V6<double> Sj = subspace(p, o);
  V6<double> vJ = zero6<double>();
  if (p.one) vJ = o.qd * Sj;
  if constexpr (BALL) {
    if (p.ball) {
      const V3<double> w = mul(R, st_ball_w(st));
      vJ = v6<double>(w, cross(oj, w));
    }
  }
  if constexpr (FREE) {
    if (p.root) vJ = v6<double>(st_vel6(st).a, z3);
  }
  double path = ks;
  o.V = path_sum<BALL>(p, vJ, sh, path, xb);
  if constexpr (FREE) {
    // gravity in the root's frame, for its whole system
    const V3<double> gr = quat_rotate_T(st_quat(st), grav);
    const int from = p.base < 0 ? 0 : p.base;
    const V3<double> t = v3<double>(__shfl(gr.x, from), __shfl(gr.y, from), __shfl(gr.z, from));
    if (p.base >= 0) gb = t;
  }
  const V6<double> cb = p.root ? zero6<double>() : crm(o.V, vJ);
  double kp = ks;
  const V6<double> A0 = path_sum<BALL>(p, cb, sh, kp, xb) - v6<double>(z3, BALL ? path * gb : gb);
  // ---- inertia, bias force
  const V3<double> Rmc = mul(R, widen<double>(p.L.mc));
  o.mc = axpy(Rmc, m, oj);
  {
    // I + [terms of the shift by o]: (2 o.Rmc + m o^2) 1 - sym(o, Rmc) ...
    const Sy3<double> J = cong(R, widen<double>(p.L.Ib));
    const double t = dot(oj, Rmc) + dot(oj, o.mc);
    o.I = sy3<double>(J.xx + t - (oj.x * Rmc.x + o.mc.x * oj.x), J.yy + t - (oj.y * Rmc.y + o.mc.y * oj.y),
                      J.zz + t - (oj.z * Rmc.z + o.mc.z * oj.z), J.xy - (oj.x * Rmc.y + o.mc.x * oj.y),
                      J.xz - (oj.x * Rmc.z + o.mc.x * oj.z), J.yz - (oj.y * Rmc.z + o.mc.y * oj.z));
  }
  LinkC<double> body;  // inertia_mul's view of it
  body.m = m;
  body.mc = o.mc;
  body.Ib = o.I;
  V6<double> F = inertia_mul(body, A0) + crf(o.V, inertia_mul(body, o.V));
  SySp<double> IA = inertia_sysp(body);
  half();
  // ---- articulated inertias and bias forces, leaves to root
  double u = 0;
  V3<double> ub = z3, yb = z3;
  o.U = zero6<double>();
  o.Di = 0;
  V3<double> tb = z3;
  if constexpr (BALL) {
    if (p.ball) tb = mul(R, ctl);
  }
  for (int d = p.maxd; d >= 0; --d) {
    if (p.dep == d) {
      for (int c = 0; c < p.cc; ++c) {
        SySp<double> Ic;
        V6<double> Fc;
        get27(xb, p.cf + c, Ic, Fc);
        IA = IA + Ic;
        F = F + Fc;
      }
      if (p.one) {
        o.U = mul(IA, Sj);
        o.Di = fast_rcp(dot(Sj, o.U));
        u = ctl.x - dot(Sj, F);
        if (p.par >= 0) put27(xb, p.lane, up(sh, rank1_down(IA, o.U, o.Di)), up(sh, F + (u * o.Di) * o.U));
      }
      if constexpr (BALL) {
        if (p.ball) {
          const SySp<double> Io = up(-oj, IA);
          o.Ai = sy3_inv(Io.A);
          o.B = Io.B;
          ub = tb - up(-oj, F).a;
          yb = mul(o.Ai, ub);
          if (p.par >= 0) {
            const M3<double> W = mul(sy_to_m3(o.Ai), o.B);
            const M3<double> BW = mul(transpose(o.B), W);
            SySp<double> Ia = zero_sysp<double>();
            Ia.C = Io.C - sy3<double>(BW.m[0], BW.m[4], BW.m[8], BW.m[1], BW.m[2], BW.m[5]);
            Ia.C = sy3<double>(ks * ks * Ia.C.xx, ks * ks * Ia.C.yy, ks * ks * Ia.C.zz, ks * ks * Ia.C.xy,
                               ks * ks * Ia.C.xz, ks * ks * Ia.C.yz);
            put27(xb, p.lane, up(sh + oj, Ia), ks * up(sh + oj, v6<double>(tb, F.l + mulT(o.B, yb))));
          }
        }
      }
    }
    wave_sync();
  }
  // ---- accelerations, root to leaves
  RootF f;
  V6<double> a = zero6<double>(), ap = zero6<double>();
  double qdd = 0;
  if constexpr (FREE) {
    if (p.root) {
      f = root_factor(IA);
      a = root_solve(f, v6<double>(-F.a, -F.l));
      const V6<double> v = st_vel6(st);
      o.abase = v6<double>(a.a, a.l - cross(v.a, v.l));
    }
  }
  for (int d = 0; d <= p.maxd; ++d) {
    if (p.dep == d) {
      if (p.par >= 0) ap = down(sh, get6(xb, 0, p.par));
      if constexpr (BALL) ap = ks * ap;
      if (p.one) {
        qdd = (u - dot(o.U, ap)) * o.Di;
        a = ap + qdd * Sj;
      }
      if constexpr (BALL) {
        if (p.ball) {
          const V3<double> lo = down(oj, ap).l, al = yb - mul(o.Ai, mul(o.B, lo));
          a = down(-oj, v6<double>(al, lo));
          o.abase.a = mulT(R, al - ap.a);  // in link coordinates, as the rate
        }
      }
      if (p.cc) put6(xb, 0, p.lane, a);
    }
    wave_sync();
  }
  o.F = mul(IA, a) + F;
  o.Ap = ap + A0 - cb;
  if constexpr (FREE) {
    if (p.root) root_pack(o, f);
  }
  if constexpr (BALL) o.R = R;
  return o;
}

// w = M^-1 r with the step's factors (r, r3, r6: the right-hand side of a
// 1-dof, ball and root lane, replaced by the solution); B: the spatial
// accelerations of the response, Bp the parent's.
template <bool FREE, bool BALL, typename S>
__device__ __forceinline__ void frame_solve(const FrameLane<S>& p, const FrameStep& o, double& r, V3<double>& r3,
                                            V6<double>& r6, V6<double>& B, V6<double>& Bp, double* xb) {
  const V6<double> Sj = subspace(p, o);
  const V3<double> sh = step_of(p, o), oj = joint_of(p, o);
  const double ks = scale_of<BALL>(p, o);
  V3<double> y3 = zero3<double>();
  for (int d = p.maxd; d >= 0; --d) {
    if (p.dep == d) {
      V6<double> s = zero6<double>();
      for (int c = 0; c < p.cc; ++c) s = s + get6(xb, 0, p.cf + c);
      if (p.one) {
        r = r - dot(Sj, s);
        if (p.par >= 0) put6(xb, 0, p.lane, up(sh, s + (r * o.Di) * o.U));
      }
      if constexpr (BALL) {
        if (p.ball) {
          y3 = mul(o.Ai, r3 - up(-oj, s).a);
          if (p.par >= 0) put6(xb, 0, p.lane, ks * up(sh + oj, v6<double>(r3, s.l + mulT(o.B, y3))));
        }
      }
      if constexpr (FREE) {
        if (p.root) r6 = r6 - s;
      }
    }
    wave_sync();
  }
  B = Bp = zero6<double>();
  if constexpr (FREE) {
    if (p.root) {
      r6 = root_solve(root_unpack(o), r6);
      B = r6;
    }
  }
  for (int d = 0; d <= p.maxd; ++d) {
    if (p.dep == d) {
      if (p.par >= 0) Bp = down(sh, get6(xb, 0, p.par));
      if constexpr (BALL) Bp = ks * Bp;
      if (p.one) {
        r = (r - dot(o.U, Bp)) * o.Di;
        B = Bp + r * Sj;
      }
      if constexpr (BALL) {
        if (p.ball) {
          const V3<double> lo = down(oj, Bp).l, al = y3 - mul(o.Ai, mul(o.B, lo));
          r3 = al - Bp.a;
          B = down(-oj, v6<double>(al, lo));
        }
      }
      if (p.cc) put6(xb, 0, p.lane, B);
    }
    wave_sync();
  }
}

// The adjoint of the step from st: x1 in, the adjoint of (q1, qd1), and out,
// that of (q, qd); returns the lane's tau_bar.  lq, lqd: the joint-limit
// torque's slopes.
template <bool FREE, bool BALL, typename S>
__device__ __forceinline__ V3<double> frame_reverse(const FrameLane<S>& p, const FrameStep& o,
                                                    const State<double, FREE>& st, double dt, double lq, double lqd,
                                                    State<double, FREE>& x1, double* xb) {
  // ---- integrator
  const double tot = x1.qd[0] + dt * x1.q[0];
  double r = dt * tot;
  V6<double> g6 = zero6<double>(), r6 = zero6<double>();
  V3<double> pb = zero3<double>(), r3 = zero3<double>(), wb = zero3<double>();
  Q4<double> qb = {0, 0, 0, 0};
  if constexpr (FREE) {
    if (p.root) {
      pb = v3<double>(x1.q[0], x1.q[1], x1.q[2]);
      qb = {x1.q[3], x1.q[4], x1.q[5], x1.q[6]};
      g6 = st_vel6(x1);
      r6 = integrate_root_adj(st_quat(st), st_vel6(st), o.abase, dt, pb, qb, g6);
    }
  }
  if constexpr (BALL) {
    if (p.ball) {
      wb = st_ball_w(x1);
      qb = quat_step_adj(st_ball_quat(st), st_ball_w(st) + dt * o.abase.a, dt, st_ball_quat(x1), wb);
      r3 = dt * mul(o.R, wb);
    }
  }
  // ---- w = M^-1 (dt qd1_bar)
  V6<double> B, Bp;
  frame_solve<FREE, BALL>(p, o, r, r3, r6, B, Bp, xb);
  // ---- <w, ID> = sum_i B_i . (I A + V x* I V): per link its share of A's
  // adjoint, I B, and of V's (the bias accelerations V_l x S_l qd_l from the
  // root to link i sum to V_i in the second), summed over subtrees.  Scaled
  // transforms don't let them: with ball joints they are taken link by link
  LinkC<double> body;
  body.m = double(p.L.m);
  body.mc = o.mc;
  body.Ib = o.I;
  V6<double> G = inertia_mul(body, B);
  V6<double> e = crmT(B, inertia_mul(body, o.V)) - inertia_mul(body, crm(o.V, B)), vJ = zero6<double>();
  if constexpr (BALL) {
    if (p.one) vJ = o.qd * subspace(p, o);
    if (p.ball) {
      const V3<double> w = mul(o.R, st_ball_w(st));
      vJ = v6<double>(w, cross(joint_of(p, o), w));
    }
  } else {
    e = e - crmT(o.V, G);
  }
  for (int d = p.maxd; d >= 0; --d) {
    if (p.dep == d) {
      for (int c = 0; c < p.cc; ++c) {
        G = G + get6(xb, 0, p.cf + c);
        e = e + get6(xb, 6, p.cf + c);
      }
      if constexpr (BALL) e = e - crmT(vJ, G);
      if (p.par >= 0) {
        const double ks = scale_of<BALL>(p, o);
        put6(xb, 0, p.lane, BALL ? ks * up(step_of(p, o), G) : up(step_of(p, o), G));
        put6(xb, 6, p.lane, BALL ? ks * up(step_of(p, o), e) : up(step_of(p, o), e));
      }
    }
    wave_sync();
  }
  // ---- the subtree turns with q: what enters it from the parent turns back
  V3<double> taub = zero3<double>();
  if (p.one) {
    const V6<double> Sj = subspace(p, o), Vp = o.V - o.qd * Sj;
    const V6<double> vb = BALL ? e : e + crmT(Vp, G);
    const double qE = dot(Sj, crf(Bp, o.F) + crf(o.Ap, G) + crf(Vp, vb));
    const double qdE = dot(Sj, crmT(o.V, G) + vb);
    x1.q[0] = x1.q[0] + qE + lq * r;
    x1.qd[0] = tot - qdE + lqd * r;
    taub.x = r;
  }
  if constexpr (BALL) {
    if (p.ball) {
      const V3<double> oj = joint_of(p, o);
      const V3<double> turn = mulT(o.R, up(-oj, crf(Bp, o.F) + crf(o.Ap, G) + crf(o.V - vJ, e)).a);
      const V3<double> rate = mulT(o.R, up(-oj, crmT(o.V, G) + e).a);
      const Q4<double> t = ball_quat_bar(st_ball_quat(st), turn);
      x1.q[0] = qb.x + t.x;
      x1.q[1] = qb.y + t.y;
      x1.q[2] = qb.z + t.z;
      x1.q[3] = qb.w + t.w;
      x1.qd[0] = wb.x - rate.x;
      x1.qd[1] = wb.y - rate.y;
      x1.qd[2] = wb.z - rate.z;
      taub = mulT(o.R, r3);
    }
  }
  if constexpr (FREE) {
    if (p.root) {
      // the root's velocity entered as [w; 0], its acceleration as qdd +
      // [0; w x v] - [0; R^T g]
      const V6<double> v = st_vel6(st);
      const Q4<double> t = quat_rot_grad(st_quat(st), widen<double>(p.g), G.l);
      const V3<double> wv = g6.a - (BALL ? e.a : e.a + crmT(o.V, G).a) - cross(v.l, G.l);
      const V3<double> lv = g6.l - cross(G.l, v.a);
      x1.q[0] = pb.x;
      x1.q[1] = pb.y;
      x1.q[2] = pb.z;
      x1.q[3] = qb.x + t.x;
      x1.q[4] = qb.y + t.y;
      x1.q[5] = qb.z + t.z;
      x1.q[6] = qb.w + t.w;
      x1.qd[0] = wv.x;
      x1.qd[1] = wv.y;
      x1.qd[2] = wv.z;
      x1.qd[3] = lv.x;
      x1.qd[4] = lv.y;
      x1.qd[5] = lv.z;
    }
  }
  return taub;
}

// A step's reverse in the backward rollout: recompute and reverse from the
// stored state and control, then tau_bar out and the trajectory's seed of x^t
// in.
template <typename S, bool FREE>
__device__ __forceinline__ void frame_outputs(const BwdArgs<S>& A, const Lane& l, int t, const V3<double>& taub,
                                              State<double, FREE>& x1, int& nonfin) {
  if (!l.active()) return;
  const S tb[3] = {S(taub.x), S(taub.y), S(taub.z)};
  const int n = l.onedof() ? 1 : l.ball() ? 3 : 0;
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (k < n) {
      A.gtau[(size_t)t * A.P.nu + l.uidx + k] = tb[k];
      nonfin += nonfinite(tb[k]);
    }
  if (A.gtraj != nullptr && t >= 1) {
    State<S, FREE> gt = {};
    const S* row = A.gtraj + (size_t)(t - 1) * (A.P.nq + A.P.nv);
    load_state(gt, l, row, row + A.P.nq);
#pragma unroll
    for (int k = 0; k < (FREE ? 7 : 1); ++k) x1.q[k] += double(gt.q[k]);
#pragma unroll
    for (int k = 0; k < (FREE ? 6 : 1); ++k) x1.qd[k] += double(gt.qd[k]);
  }
}
template <typename S, bool FREE, int FR>
__device__ __forceinline__ void frame_step(const BwdArgs<S>& A, const Lane& l, const FrameLane<S>& p, double* xb,
                                           const State<S, FREE>& st, const V3<S>& tau, int t, State<double, FREE>& x1,
                                           int& nonfin) {
  constexpr bool BALL = FREE && FR == kFrBall;
  const State<double, FREE> sr = cvt_state<double>(st);
  const FrameStep o = frame_recompute<FREE, BALL>(p, sr, limit_tau<FR>(A.P, l, sr, cvt3<double>(tau)), xb);
  double lq, lqd;
  limit_slopes<FR>(A.P, l, sr, lq, lqd);
  const V3<double> taub = frame_reverse<FREE, BALL>(p, o, sr, double(A.dt), lq, lqd, x1, xb);
  frame_outputs<S, FREE>(A, l, t, taub, x1, nonfin);
}

// A step's record in LDS, [field][lane]: what the reverse reads of a recompute.
template <bool FREE, bool BALL>
constexpr int kFrameTape = 42 + (FREE ? 6 : 0) + (BALL ? 24 : 0);
template <bool FREE, bool BALL, typename F>
__device__ __forceinline__ void frame_fields(FrameStep& o, F&& f) {
  int k = 0;
  auto w = [&](double& x) { f(k++, x); };
  auto w3 = [&](V3<double>& v) { w(v.x); w(v.y); w(v.z); };
  auto w6 = [&](V6<double>& v) { w3(v.a); w3(v.l); };
  auto ws = [&](Sy3<double>& m) { w(m.xx); w(m.yy); w(m.zz); w(m.xy); w(m.xz); w(m.yz); };
  w3(o.ax); w3(o.at); w6(o.U); w6(o.V); w6(o.Ap); w6(o.F);
  w(o.Di);
  w3(o.mc);
  ws(o.I);
  w(o.q);
  w(o.qd);
  if constexpr (FREE) w6(o.abase);
  if constexpr (BALL) {
#pragma unroll
    for (int j = 0; j < 9; ++j) w(o.R.m[j]);
#pragma unroll
    for (int j = 0; j < 9; ++j) w(o.B.m[j]);
    ws(o.Ai);
  }
}

// The wavefronts of the pipelined backward on one batch, and its LDS: NR
// replaying (K > 1), NP recomputing, one reversing.
template <typename S, bool FREE, int FR, int NP, int NR>
struct FramePipe {
  static constexpr bool BALL = FREE && FR == kFrBall;
  static constexpr int waves = NR + NP + 1;
  static constexpr int TW = kFrameTape<FREE, BALL> * kWave;
  static constexpr size_t rec = XB * kWave;  // one exchange buffer
  // numbers of a replayed state in the ring (slots, then mfree extended ones)
  static __host__ __device__ int state(int mfree) { return 2 * kWave + 11 * mfree; }
  static __host__ __device__ size_t lds(int K, int mfree) {
    return (size_t)(2 * TW + (NP + 1) * rec) * sizeof(double) + NR * ((size_t)3 * K * state(mfree) + rec) * sizeof(S);
  }
};

// Pipelined backward rollout, K >= 1, in time slots ended by a workgroup
// barrier, one reversed step a slot.  The recomputes do not depend on one
// another: with NP producers a step's recompute takes NP slots (with two, a
// barrier after the velocities and inertias, which is about half of it), the last of them the one before its reverse, and only that
// one writes the step's record, so that two records are enough.  K > 1 (NR =
// 1): one more wavefront replays the segment before, a step a slot, into a
// ring of three segments of states in LDS (one replayed, one recomputed, the
// last steps of one still to be reversed), so that a segment costs its slowest
// part and not replay, recompute and reverse in turn.  The reversing wavefront
// bounds K == 1, the replaying one K > 1.  Adjoints, one wavefront / one
// producer / two: 1024 quadrupeds x 200 steps in segments of 10, 2.86 / 1.24 /
// 1.16 ms; 1024 ball-jointed ones x 100 steps, K = 1, 1.22 / 0.70 / 0.60.
// CHAIN: the replay takes the register exchange of the chain kernels, as the
// rollout did.
template <typename S, bool FREE, int FR, bool CHAIN, int NP, int NR>
__global__ __launch_bounds__((NP + NR + 1) * kWave)
__attribute__((amdgpu_waves_per_eu(FREE ? 1 : 2))) void k_backward_frame_pipe(BwdArgs<S> A) {
  using P = FramePipe<S, FREE, FR, NP, NR>;
  constexpr bool BALL = P::BALL;
  static_assert(NP == 1 || NP == 2, "one barrier half way");
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  double* const tape = lds<double>();
  double* const xbs = tape + 2 * P::TW;
  S* const xreplay = reinterpret_cast<S*>(xbs + (NP + 1) * P::rec);
  S* const ring = xreplay + P::rec;
  const int wb = blockIdx.x;
  const Lane l = load_lane(A.P, wb);
  const int maxd = wave_maxd(A.P, wb);
  const int ns = A.P.nslots, nu = A.P.nu, nf = A.P.nfree, mf = A.P.mfree, T = A.T;
  const size_t RW = state_record(ns, nf);
  const bool act = l.active();
  // K > 1: segments last to first, and in each its steps; the first one may be
  // short of seg.  K == 1: one segment of T steps
  const int seg = NR ? A.K : T, nseg = (T + seg - 1) / seg, steps = nseg * seg;
  const int ahead = (NR ? seg : 0) + NP, slots = steps + ahead;  // step n is reversed in slot n + ahead
  const unsigned long long extended = __ballot(l.fidx >= 0);
  const int rl = l.fidx < 0 ? -1 : __popcll(extended & ((1ull << l.lane) - 1));
  const int sw = P::state(mf);
  auto length = [&](int c) { return min(seg, T - (nseg - 1 - c) * seg); };  // of the c-th segment
  auto has = [&](int n) { return n < steps && n % seg < length(n / seg); };
  auto time_of = [&](int n) { return (nseg - 1 - n / seg) * seg + length(n / seg) - 1 - n % seg; };
  auto get = [&](int n, State<S, FREE>& st) {
    if (!act) return;
    const int c = n / seg;
    if constexpr (NR > 0) get_slot(st, ring + (size_t)((c % 3) * seg + length(c) - 1 - n % seg) * sw, kWave, mf, l.lane, rl);
    else get_slot(st, A.ck + (size_t)time_of(n) * RW, ns, nf, l.slot, l.fidx);
  };
  int slot = 0;
  auto next_slot = [&] {
    __syncthreads();
    ++slot;
  };
  if (NR > 0 && wid < NR) {
    const LinkC<S> L = load_linkc<S, FR>(A.P, l);
    State<S, FREE> st = {};
    while (slot < slots) {
      const int c = slot / seg, i = slot % seg;
      if (c < nseg) {
        const int t0 = (nseg - 1 - c) * seg;
        S* const base = ring + (size_t)(c % 3) * seg * sw;
        if (i == 0 && act) {
          get_slot(st, A.ck + (size_t)(nseg - 1 - c) * RW, ns, nf, l.slot, l.fidx);
          put_slot(st, base, kWave, mf, l.lane, rl);
        }
        if (i + 1 < length(c)) {
          const V3<S> tau = act ? load_ctl<BALL>(A.tau + (size_t)(t0 + i) * nu, l) : zero3<S>();
          advance<FR, CHAIN, false>(A.P, gravity(A.P), l, L, st, tau, A.dt, maxd, xreplay);
          if (act) put_slot(st, base + (size_t)(i + 1) * sw, kWave, mf, l.lane, rl);
        }
      }
      next_slot();
    }
  } else if (wid < NR + NP) {
    const int j = wid - NR;
    double* const xb = xbs + j * P::rec;
    const FrameLane<S> p = frame_lane<S, FR>(A.P, l, maxd);
    State<S, FREE> nxt = {};
    V3<S> nt = zero3<S>();
    auto fetch = [&](int n) {
      if (!has(n)) return;
      if constexpr (NR == 0) get(n, nxt);
      if (act) nt = load_ctl<BALL>(A.tau + (size_t)time_of(n) * nu, l);
    };
    fetch(j);
    for (int n = j; n < steps; n += NP) {
      while (slot < n + ahead - NP) next_slot();
      if (has(n)) {
        if constexpr (NR > 0) get(n, nxt);
        const State<double, FREE> st = cvt_state<double>(nxt);
        const V3<double> tau = cvt3<double>(nt);
        fetch(n + NP);
        FrameStep o = frame_recompute<FREE, BALL>(p, st, limit_tau<FR>(A.P, l, st, tau), xb, [&] {
          if constexpr (NP == 2) next_slot();
        });
        double* const tp = tape + (n & 1) * P::TW;
        frame_fields<FREE, BALL>(o, [&](int f, double& v) { tp[f * kWave + l.lane] = v; });
      } else {
        fetch(n + NP);
      }
    }
    while (slot < slots) next_slot();
  } else {
    double* const xb = xbs + NP * P::rec;
    const FrameLane<S> p = frame_lane<S, FR>(A.P, l, maxd);
    const double dt = double(A.dt);
    int nonfin = 0;
    State<double, FREE> x1 = seed_state<S, double, FREE>(A, l);
    State<S, FREE> nxt = {};
    if constexpr (FREE && NR == 0) get(0, nxt);
    while (slot < ahead) next_slot();
    for (int n = 0; n < steps; ++n) {
      if (has(n)) {
        FrameStep o;
        const double* tp = tape + (n & 1) * P::TW;
        frame_fields<FREE, BALL>(o, [&](int f, double& v) { v = tp[f * kWave + l.lane]; });
        State<double, FREE> st = {};
        if constexpr (FREE) {
          if constexpr (NR > 0) get(n, nxt);
          st = cvt_state<double>(nxt);
          if (NR == 0 && has(n + 1)) get(n + 1, nxt);
        } else {
          st.q[0] = o.q;
          st.qd[0] = o.qd;
        }
        double lq, lqd;
        limit_slopes<FR>(A.P, l, st, lq, lqd);
        const V3<double> taub = frame_reverse<FREE, BALL>(p, o, st, dt, lq, lqd, x1, xb);
        frame_outputs<S, FREE>(A, l, time_of(n), taub, x1, nonfin);
      }
      next_slot();
    }
    if (act) {
      const State<S, FREE> x0 = cvt_state<S>(x1);
      store_state(x0, l, A.gq0, A.gqd0);
      nonfin += nonfinite_state(x0, l);
    }
    report_nonfinite(A.P.status, nonfin);
  }
}

}  // namespace

}  // namespace aba
