// Rollouts with contact and their gradient on the GPU: 16 lanes per system,
// four systems per wavefront, one wavefront per workgroup.
//
// What bounds these kernels is a step's serial chain, not its arithmetic: 60
// Gauss-Seidel sweeps of up to 12 dependent rows, and the tree recursions.
// So a system's independent work is spread over the 16 lanes of one DPP row
// and every shared quantity sits in LDS:
//   - lane i holds link i (links in breadth-first order, the root in lane 0)
//     in the tree recursions;
//   - lane r < 12 holds contact row r = 3 k + d (sphere k; d = 0 the normal
//     e_y, 1 and 2 the tangents e_x, e_z): its row of A, its bounds and its
//     impulse stay in registers through both solves, and a row's new impulse
//     reaches the other lanes by a DPP row broadcast;
//   - the degrees of freedom are numbered as they are eliminated: the free
//     root's six (in the root's own frame), then one per 1-dof link.
// All spatial quantities are taken about one origin in one frame, the base
// frame: the world for a fixed base, the root link's own frame for a free
// root (so the root's motion subspace is the identity), its origin at the
// root link's; of where that stands only the height enters, through the gaps.
// A tree recursion then adds 6-vectors and transforms nothing.  An inertia
// about a far origin holds the squared distance, of which a joint's share is
// the small remainder: in FP64 (OWN) the articulated inertias and bias forces
// are therefore taken about each link's own joint's origin and shifted from
// link to link, and only U = I^A S comes back to the common one.  One free step
// of a quadruped in FP64, error of qd1 / tau_bar: one lane per system in link
// frames 1.0e-16 / 2.1e-16, one origin 8.5e-16 / 1.7e-15, own 1.3e-16 / 3.9e-16.
//
// Arithmetic is FP64 for both dtypes; the state is rounded to the dtype S
// after every step, so the gradient, recomputed from the stored states, is
// that of the map the rollout applied.
//
// The step's contact system without M^-1 J^T: with M = L^T D L of the
// articulated-body recursion (L_ij = U_i . S_j / D_i for j an ancestor of i),
// A = J M^-1 J^T = Z^T D^-1 Z, Z = L^-T J^T, and a column of Z is supported
// on its contact's path to the root.  Only the gradient forms M^-1 J^T.
//
// Measured on 4096 standing quadrupeds (3 feet down on average, 30 sweeps per
// solve, FP32 states): a rollout step 30 us (590 us with one lane per system
// and its records in LDS), a gradient step 107 us (3.1 ms, records in private
// memory); of these the sweeps are 11 and 30 us.  250 systems in FP64: 26 us
// and 60 us, by the kernel of two wavefronts per four systems (520 us and
// 2.5 ms).
#pragma once

#include <utility>

#include "aba_lane.h"
#include "contact_step.h"

namespace aba_contact {

using aba::M3;
using aba::Q4;
using aba::Sy3;
using aba::SySp;
using aba::V3;
using aba::V6;

constexpr int kGrp = 16;      // lanes per system
constexpr int kSysWave = 4;   // systems per wavefront
constexpr int kRec = 28;      // doubles per lane of the exchange region
constexpr int kLk = 15;       // doubles per link record: S 6, U/D 6, 1/D, qd_minus, g
constexpr int kRt = 34;       // root record: L 15, 1/D 6, qd_minus 6, g 6

// The model in lane order, and the LDS layout of one system (in doubles).
struct WTopo {
  int n, nq, nv, nu, nc, niter;
  int free_root, maxd, dd;  // dd: degrees of freedom on the longest path
  int link[kGrp], par[kGrp], dep[kGrp], cf[kGrp], ccn[kGrp], jt[kGrp], qi[kGrp], vi[kGrp], ui[kGrp];
  int sub[kGrp];            // bit i: lane i is in the subtree
  int sph[kGrp];            // bit k: sphere k is on a link of the subtree
  int cl[kNC];              // sphere's link lane
  int com[kNC][kNC];        // degrees of freedom common to two spheres' paths
  double mu, beta, g[3];
  int has_limits;
  double lim[kGrp][4];
  int oRT, oJ, oZ, oW, oX, stride;
};

// Fills the lane order and the layout from the model (links in topological
// order, parent before child); grad: with the gradient's regions.
inline WTopo make_wave_topo(const CTopo& tp, bool grad) {
  WTopo w{};
  w.n = tp.n;
  w.nq = tp.nq;
  w.nv = tp.nv;
  w.nu = tp.nu;
  w.nc = tp.nc;
  w.niter = tp.niter;
  w.free_root = tp.jtype[0] == SIM_JOINT_FREE;
  w.mu = tp.mu;
  w.beta = tp.beta;
  for (int k = 0; k < 3; ++k) w.g[k] = tp.g[k];
  w.has_limits = tp.has_limits;
  int lane_of[kNL];
  int m = 0;
  w.link[m] = 0;
  lane_of[0] = m++;
  for (int i = 0; i < m; ++i) {  // breadth first: a link's children take consecutive lanes
    w.cf[i] = m;
    for (int j = 1; j < tp.n; ++j)
      if (tp.parent[j] == w.link[i]) {
        w.link[m] = j;
        lane_of[j] = m++;
      }
    w.ccn[i] = m - w.cf[i];
  }
  for (int i = 0; i < kGrp; ++i) {
    if (i >= tp.n) {
      w.jt[i] = -1;
      w.par[i] = -1;
      w.dep[i] = -1;
      continue;
    }
    const int l = w.link[i];
    w.jt[i] = tp.jtype[l];
    w.par[i] = tp.parent[l] < 0 ? -1 : lane_of[tp.parent[l]];
    w.dep[i] = w.par[i] < 0 ? 0 : w.dep[w.par[i]] + 1;
    w.maxd = w.dep[i] > w.maxd ? w.dep[i] : w.maxd;
    w.qi[i] = tp.qi[l];
    w.vi[i] = tp.vi[l];
    w.ui[i] = tp.ui[l];
    for (int k = 0; k < 4; ++k) w.lim[i][k] = tp.lim[l][k];
    for (int j = i; j >= 0; j = w.par[j]) w.sub[j] |= 1 << i;
  }
  w.dd = w.maxd + 1 + (w.free_root ? 5 : 0);
  for (int k = 0; k < tp.nc; ++k) {
    w.cl[k] = lane_of[tp.clink[k]];
    for (int j = w.cl[k]; j >= 0; j = w.par[j]) w.sph[j] |= 1 << k;
  }
  for (int k = 0; k < tp.nc; ++k)
    for (int c = 0; c < tp.nc; ++c) {
      int a = w.cl[k], b = w.cl[c];
      while (a != b && a >= 0 && b >= 0) {
        if (w.dep[a] >= w.dep[b]) a = w.par[a];
        else b = w.par[b];
      }
      w.com[k][c] = (a == b && a >= 0) ? w.dep[a] + 1 + (w.free_root ? 5 : 0) : 0;
    }
  w.oRT = kLk * tp.n;
  w.oJ = w.oRT + kRt;
  w.oZ = w.oJ + kNR * w.dd;
  w.oW = w.oZ + kNR * w.dd;
  w.oX = w.oW + (grad ? kNR * tp.nv : 0);
  w.oX += w.oX & 1;  // 16-byte aligned records
  int x = kRec * kGrp;
  if (grad) {
    const int sweeps = kGrp * (tp.niter + 1);
    const int stage = kNR * kNR + 2 * tp.nv + 6 * kGrp + tp.nv * w.dd;
    x = sweeps > x ? sweeps : x;
    x = stage > x ? stage : x;
  }
  w.stride = w.oX + x;
  w.stride += w.stride & 1;
  return w;
}
inline size_t wave_lds_bytes(const WTopo& w) { return (size_t)w.stride * kSysWave * sizeof(double); }

#if defined(__HIPCC__)

namespace wave {

using D = double;

__device__ __forceinline__ void sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// the value of lane J of the row of 16 (every lane active)
template <int J>
__device__ __forceinline__ D bc(D x) {
  return __builtin_amdgcn_update_dpp(0.0, x, 0x150 + J, 0xf, 0xf, true);
}
template <int N>
__device__ __forceinline__ D ror(D x) {
  return __builtin_amdgcn_update_dpp(0.0, x, 0x120 + N, 0xf, 0xf, true);
}
// sum, and largest, over the 16 lanes of a row
__device__ __forceinline__ D rsum(D x) {
  x += ror<8>(x);
  x += ror<4>(x);
  x += ror<2>(x);
  return x + ror<1>(x);
}
__device__ __forceinline__ D rmax(D x) {
  D y = ror<8>(x);
  x = y > x ? y : x;
  y = ror<4>(x);
  x = y > x ? y : x;
  y = ror<2>(x);
  x = y > x ? y : x;
  y = ror<1>(x);
  return y > x ? y : x;
}
template <int N, typename F>
__device__ __forceinline__ void unroll(F&& f) {
  [&]<int... I>(std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
  (std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ V3<D> ld3(const D* p) { return aba::v3<D>(p[0], p[1], p[2]); }
__device__ __forceinline__ V6<D> ld6(const D* p) { return aba::v6<D>(ld3(p), ld3(p + 3)); }
__device__ __forceinline__ void st3(D* p, const V3<D>& v) {
  p[0] = v.x;
  p[1] = v.y;
  p[2] = v.z;
}
__device__ __forceinline__ void st6(D* p, const V6<D>& v) {
  st3(p, v.a);
  st3(p + 3, v.l);
}
__device__ __forceinline__ M3<D> ld9(const D* p) {
  M3<D> M;
#pragma unroll
  for (int k = 0; k < 9; ++k) M.m[k] = p[k];
  return M;
}
__device__ __forceinline__ void st21(D* p, const SySp<D>& M) {
  const D v[21] = {M.A.xx,   M.A.yy,   M.A.zz,   M.A.xy,   M.A.xz,   M.A.yz,   M.B.m[0],
                   M.B.m[1], M.B.m[2], M.B.m[3], M.B.m[4], M.B.m[5], M.B.m[6], M.B.m[7],
                   M.B.m[8], M.C.xx,   M.C.yy,   M.C.zz,   M.C.xy,   M.C.xz,   M.C.yz};
#pragma unroll
  for (int k = 0; k < 21; ++k) p[k] = v[k];
}
__device__ __forceinline__ SySp<D> ld21(const D* p) {
  SySp<D> M;
  M.A = aba::sy3<D>(p[0], p[1], p[2], p[3], p[4], p[5]);
#pragma unroll
  for (int k = 0; k < 9; ++k) M.B.m[k] = p[6 + k];
  M.C = aba::sy3<D>(p[15], p[16], p[17], p[18], p[19], p[20]);
  return M;
}
__device__ __forceinline__ D comp(const V6<D>& v, int e) {
  return e == 0 ? v.a.x : e == 1 ? v.a.y : e == 2 ? v.a.z : e == 3 ? v.l.x : e == 4 ? v.l.y : v.l.z;
}

// A rigid body's spatial inertia about the base origin: mass, first moment,
// second moment.
struct Body {
  D m;
  V3<D> mc;
  Sy3<D> I;
};
__device__ __forceinline__ V6<D> mul(const Body& b, const V6<D>& v) {
  return aba::v6<D>(aba::mul(b.I, v.a) + cross(b.mc, v.l), b.m * v.l - cross(b.mc, v.a));
}

// From one origin to another, d the step from the first to the second: a
// motion goes down it, a force and an inertia come up.
__device__ __forceinline__ V6<D> down(const V3<D>& d, const V6<D>& v) { return aba::v6<D>(v.a, v.l + cross(v.a, d)); }
__device__ __forceinline__ V6<D> up(const V3<D>& d, const V6<D>& f) { return aba::v6<D>(f.a + cross(d, f.l), f.l); }
__device__ __forceinline__ SySp<D> up(const V3<D>& d, const SySp<D>& M) {
  M3<D> E;
#pragma unroll
  for (int k = 0; k < 9; ++k) E.m[k] = k % 4 == 0 ? 1.0 : 0.0;
  return aba::congruence_XT(E, d, M);
}

// The rotation nearest to R by a Newton step, R (3 - R^T R) / 2: the gradient
// takes every pose for a rotation, and a joint frame in FP32 is one only to
// 6e-8 (two steps, once a launch: of matrices with a few digits, too).  Error of
// tau_bar, one step of 8 to 16 links in contact, FP32: 1e-7 -> 4e-8.
__device__ __forceinline__ M3<D> nearest_rotation(const M3<D>& R) {
  M3<D> G = aba::mul(aba::transpose(R), R);
#pragma unroll
  for (int k = 0; k < 9; ++k) G.m[k] = (k % 4 == 0 ? 1.5 : 0.0) - 0.5 * G.m[k];
  return aba::mul(R, G);
}

// One lane's constants: its link, and its contact row.
struct Lane {
  int gl, p, dep, cf, ccn, jt, slot, dof, sub, sph;
  int qi, vi, ui;
  bool one, root;  // a 1-dof link; the free root
  M3<D> ETt;       // joint frame -> parent
  V3<D> rT, ax, com;
  D m;
  Sy3<D> Ic;
  D lo, hi, lk, ld;  // joint limits
  int k, d;          // sphere and direction of the row (k = -1: no such row)
  int cl, nc4[kNC];
  V3<D> cc;
  D rad;
};

template <typename S>
__device__ __forceinline__ Lane load_lane(const WTopo& tp, const S* P, size_t B, int s) {
  Lane l;
  l.gl = threadIdx.x % kGrp;
  const int i = l.gl;
  l.p = tp.par[i];
  l.dep = tp.dep[i];
  l.cf = tp.cf[i];
  l.ccn = tp.ccn[i];
  l.jt = tp.jt[i];
  l.sub = tp.sub[i];
  l.sph = tp.sph[i];
  l.qi = tp.qi[i];
  l.vi = tp.vi[i];
  l.ui = tp.ui[i];
  const int off = tp.free_root ? 5 : 0;
  l.slot = l.dep + off;
  l.dof = i + off;
  l.root = l.jt == SIM_JOINT_FREE;
  l.one = l.jt >= 0 && !l.root;
  const int pb = kParLink * tp.link[i < tp.n ? i : 0];
  auto at = [&](int k) { return D(P[(size_t)(pb + k) * B + s]); };
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) l.ETt.m[3 * b + a] = at(3 * a + b);
  if (l.one) l.ETt = nearest_rotation(nearest_rotation(l.ETt));
  l.rT = aba::v3<D>(at(9), at(10), at(11));
  l.ax = aba::v3<D>(at(12), at(13), at(14));
  if (l.one) l.ax = (1.0 / sqrt(dot(l.ax, l.ax))) * l.ax;
  l.m = at(15);
  l.com = aba::v3<D>(at(16), at(17), at(18));
  l.Ic = aba::sy3<D>(at(19), at(20), at(21), at(22), at(23), at(24));
  l.lo = tp.lim[i][0];
  l.hi = tp.lim[i][1];
  l.lk = tp.lim[i][2];
  l.ld = tp.lim[i][3];
  l.k = i < kNR && i / 3 < tp.nc ? i / 3 : -1;
  l.d = i % 3;
  const int k = l.k < 0 ? 0 : l.k;
  l.cl = l.k < 0 ? -1 : tp.cl[k];
#pragma unroll
  for (int c = 0; c < kNC; ++c) l.nc4[c] = l.k < 0 ? 0 : tp.com[k][c];
  l.cc = aba::zero3<D>();
  l.rad = 0;
  if (l.k >= 0) {
    const int sb = kParLink * tp.n + kParSphere * k;
    auto as = [&](int e) { return D(P[(size_t)(sb + e) * B + s]); };
    l.cc = aba::v3<D>(as(0), as(1), as(2));
    l.rad = as(3);
  }
  return l;
}

constexpr int kStateNumbers = 15;
// Per-lane state: a 1-dof link's q, qd; the root's pose and body velocity.
struct State {
  D q, qd;
  V3<D> pos;
  Q4<D> quat;
  V6<D> vel;
};
template <typename S>
__device__ __forceinline__ void load_state(State& x, const Lane& l, const S* q, const S* qd, size_t B, int s) {
  if (l.one) {
    x.q = D(q[l.qi * B + s]);
    x.qd = D(qd[l.vi * B + s]);
  }
  if (l.root) {
    auto at = [&](int k) { return D(q[(l.qi + k) * B + s]); };
    auto av = [&](int k) { return D(qd[(l.vi + k) * B + s]); };
    x.pos = aba::v3<D>(at(0), at(1), at(2));
    x.quat = {at(3), at(4), at(5), at(6)};
    x.vel = aba::v6<D>(aba::v3<D>(av(0), av(1), av(2)), aba::v3<D>(av(3), av(4), av(5)));
  }
}
template <typename S>
__device__ __forceinline__ void store_state(const State& x, const Lane& l, S* q, S* qd, size_t B, int s) {
  if (l.one) {
    q[l.qi * B + s] = S(x.q);
    qd[l.vi * B + s] = S(x.qd);
  }
  if (l.root) {
    const D a[7] = {x.pos.x, x.pos.y, x.pos.z, x.quat.x, x.quat.y, x.quat.z, x.quat.w};
    const D b[6] = {x.vel.a.x, x.vel.a.y, x.vel.a.z, x.vel.l.x, x.vel.l.y, x.vel.l.z};
#pragma unroll
    for (int k = 0; k < 7; ++k) q[(l.qi + k) * B + s] = S(a[k]);
#pragma unroll
    for (int k = 0; k < 6; ++k) qd[(l.vi + k) * B + s] = S(b[k]);
  }
}
// the state's numbers in turn
template <typename F>
__device__ __forceinline__ void each(State& x, F&& f) {
  D* const v[kStateNumbers] = {&x.q,      &x.qd,     &x.pos.x,  &x.pos.y,   &x.pos.z,   &x.quat.x,  &x.quat.y, &x.quat.z,
                               &x.quat.w, &x.vel.a.x, &x.vel.a.y, &x.vel.a.z, &x.vel.l.x, &x.vel.l.y, &x.vel.l.z};
#pragma unroll
  for (int k = 0; k < kStateNumbers; ++k) f(k, *v[k]);
}
__device__ __forceinline__ State zero_state() {
  State x;
  x.q = x.qd = 0;
  x.pos = aba::zero3<D>();
  x.quat = {0, 0, 0, 1};
  x.vel = aba::zero6<D>();
  return x;
}
// every number as the dtype holds it
template <typename S>
__device__ __forceinline__ void round_state(State& x) {
  auto r = [](D v) { return D(S(v)); };
  x.q = r(x.q);
  x.qd = r(x.qd);
  x.pos = aba::v3<D>(r(x.pos.x), r(x.pos.y), r(x.pos.z));
  x.quat = {r(x.quat.x), r(x.quat.y), r(x.quat.z), r(x.quat.w)};
  x.vel = aba::v6<D>(aba::v3<D>(r(x.vel.a.x), r(x.vel.a.y), r(x.vel.a.z)),
                     aba::v3<D>(r(x.vel.l.x), r(x.vel.l.y), r(x.vel.l.z)));
}

// The group's LDS.
struct Lds {
  D *lk, *rt, *J, *Z, *W, *X;
  const int* meta;  // per lane: parent (-1 = none) << 8 | slot << 1 | prismatic
};
__device__ __forceinline__ Lds lds_of(const WTopo& tp, D* base, const int* meta) {
  D* g = base + (size_t)(threadIdx.x / kGrp) * tp.stride;
  return {g, g + tp.oRT, g + tp.oJ, g + tp.oZ, g + tp.oW, g + tp.oX, meta};
}
__device__ __forceinline__ void fill_meta(const WTopo& tp, int* meta) {
  if (threadIdx.x < kGrp) {
    const int i = threadIdx.x;
    const int slot = tp.dep[i] + (tp.free_root ? 5 : 0);
    // the path walks stop at the free root
    const int p = tp.par[i] >= 0 && !(tp.free_root && tp.par[i] == 0) ? tp.par[i] : -1;
    meta[i] = (p + 1) << 8 | (slot & 0x7f) << 1 | (tp.jt[i] == SIM_JOINT_PRISMATIC);
  }
}
__device__ __forceinline__ int meta_par(int m) { return (m >> 8) - 1; }
__device__ __forceinline__ int meta_slot(int m) { return (m >> 1) & 0x7f; }
// lane of a row's contact link for a walk along its 1-dof links (-1: none)
__device__ __forceinline__ int walk_start(const WTopo& tp, const Lane& l) {
  return tp.free_root && l.cl == 0 ? -1 : l.cl;
}

// What a step leaves in a lane.
struct Step {
  V6<D> S, V, A0, U, a, h;  // subspace, velocity, bias acceleration, I^A S, acceleration beyond A0, I V
  Body I;
  D Dinv, qdd, qdm, qd1, y;
  V6<D> qdm6, qd16, y6;     // the free root's
  // contact row
  Q4<D> quat;               // the root's, in every lane
  D s;                      // its squared length
  V3<D> n, ny, pt, cb;
  V6<D> Phi;
  D phi, dinv, b, x, lamn;
  D A[kNR];
  unsigned long long clo1, chi1, clo2, chi2;  // clamped sweeps of the two solves
  bool act;
  int any;  // bit k: sphere k is active in some system of the wavefront
  int na;
};

// The free root's six degrees of freedom, eliminated last to first:
// r = L0^-T r in place.
__device__ __forceinline__ void root_up(const D* rt, D (&r)[6]) {
#pragma unroll
  for (int e = 5; e >= 0; --e)
#pragma unroll
    for (int i = 0; i < e; ++i) r[i] = fma(-rt[e * (e - 1) / 2 + i], r[e], r[i]);
}
// x = L0^-1 D0^-1 r
__device__ __forceinline__ void root_down(const D* rt, D (&r)[6]) {
#pragma unroll
  for (int e = 0; e < 6; ++e) {
    D v = r[e] * rt[15 + e];
#pragma unroll
    for (int i = 0; i < e; ++i) v = fma(-rt[e * (e - 1) / 2 + i], r[i], v);
    r[e] = v;
  }
}
__device__ __forceinline__ V6<D> to6(const D (&r)[6]) {
  return aba::v6<D>(aba::v3<D>(r[0], r[1], r[2]), aba::v3<D>(r[3], r[4], r[5]));
}
__device__ __forceinline__ void from6(const V6<D>& v, D (&r)[6]) {
  r[0] = v.a.x; r[1] = v.a.y; r[2] = v.a.z; r[3] = v.l.x; r[4] = v.l.y; r[5] = v.l.z;
}

// Root to leaves: accelerations from the eliminated right-hand side u (the
// root's: a0).  Returns the link's joint acceleration; a: its spatial one.
__device__ __forceinline__ D down(const WTopo& tp, const Lane& l, const Lds& g, const Step& o, D u, const V6<D>& a0,
                                  V6<D>& a) {
  D qdd = 0;
  a = l.root ? a0 : aba::zero6<D>();
  for (int d = 0; d <= tp.maxd; ++d) {
    if (l.dep == d) {
      if (l.one) {
        const V6<D> ap = l.p >= 0 ? ld6(g.X + l.p * kRec) : aba::zero6<D>();
        qdd = (u - dot(o.U, ap)) * o.Dinv;
        a = ap + qdd * o.S;
      }
      if (l.ccn) st6(g.X + l.gl * kRec, a);
    }
    sync();
  }
  return qdd;
}
// Leaves to root: eliminates the right-hand side r (r6 the root's) in place.
__device__ __forceinline__ void up(const WTopo& tp, const Lane& l, const Lds& g, const Step& o, D& r, V6<D>& r6) {
  for (int d = tp.maxd; d >= 0; --d) {
    if (l.dep == d) {
      V6<D> p = aba::zero6<D>();
      for (int c = 0; c < l.ccn; ++c) p = p + ld6(g.X + (l.cf + c) * kRec);
      if (l.one) {
        r = r - dot(o.S, p);
        if (l.p >= 0) st6(g.X + l.gl * kRec, p + (r * o.Dinv) * o.U);
      } else {
        r6 = r6 - p;
      }
    }
    sync();
  }
}
// M^-1 applied to (r, r6); a: the spatial accelerations of the response.
__device__ __forceinline__ void minv(const WTopo& tp, const Lane& l, const Lds& g, const Step& o, D& r, V6<D>& r6,
                                     V6<D>& a) {
  up(tp, l, g, o, r, r6);
  V6<D> a0 = aba::zero6<D>();
  if (tp.free_root && l.root) {
    D t[6];
    from6(r6, t);
    root_up(g.rt, t);
    root_down(g.rt, t);
    a0 = to6(t);
  }
  r6 = a0;
  r = down(tp, l, g, o, r, a0, a);
}

// Projected Gauss-Seidel from zero: niter sweeps over the rows of the active
// spheres (ROWS = 1: their normal rows only).  Lane r keeps row r of A (the
// diagonal entry zero) and the running sum acc = b_r + sum_j A_rj x_j, begun
// anew after the lane's own row: row j's new value reaches it by broadcast
// and enters once per sweep, so the sum is the one a row by row evaluation
// forms.  REC: the start of every sweep and the result go to sw, the
// clamped sweeps to clo and chi.
template <int ROWS, bool REC>
__device__ __forceinline__ D sweeps(const Lane& l, const Step& o, D dinv, D lo, D hi, int niter, D* sw, int ld,
                                    unsigned long long& clo, unsigned long long& chi) {
  D acc = o.b, x = 0;
  const bool mine = l.k >= 0 && (ROWS == 3 || l.d == 0);
  D* const my = sw + (ROWS == 3 ? l.gl : l.k);
  if (REC) clo = chi = 0;
  for (int it = 0; it < niter; ++it) {
    if (REC && mine) my[it * ld] = x;
    D yl = 0;
    unroll<kNC>([&](auto K) {
      if (o.any >> K & 1) {
        unroll<ROWS>([&](auto R) {
          constexpr int j = 3 * K + R;
          const D y = -(acc * dinv);
          D xn = y < lo ? lo : y;
          xn = xn > hi ? hi : xn;
          const D xj = bc<j>(xn);
          const bool own = l.gl == j;
          if (REC) yl = own ? y : yl;
          x = own ? xn : x;
          acc = fma(o.A[j], xj, own ? o.b : acc);
        });
      }
    });
    if (REC) {
      clo |= (unsigned long long)(yl < lo) << it;
      chi |= (unsigned long long)(yl > hi) << it;
    }
  }
  if (REC && mine) my[niter * ld] = x;
  return x;
}

// One step from x under the link's control u.  REC: records the sweeps and
// keeps what the adjoint needs.  OWN: FP64 states (above).
template <bool REC, bool OWN>
__device__ __forceinline__ void step(const WTopo& tp, const Lane& l, const Lds& g, const State& x, D u, D dt, D mu,
                                     Step& o) {
  const V3<D> grav = aba::v3<D>(tp.g[0], tp.g[1], tp.g[2]);
  const V3<D> z3 = aba::zero3<D>();
  o.quat = {bc<0>(x.quat.x), bc<0>(x.quat.y), bc<0>(x.quat.z), bc<0>(x.quat.w)};
  // ---- poses, velocities, bias accelerations, root to leaves
  M3<D> R;
  V3<D> org = z3, sh = z3;  // sh: the step from the parent's origin, to be shifted by
#pragma unroll
  for (int k = 0; k < 9; ++k) R.m[k] = k % 4 == 0 ? 1.0 : 0.0;
  const V3<D> gb = tp.free_root ? quat_rotate_T(o.quat, grav) : grav;
  o.S = o.U = aba::zero6<D>();
  // a free root: the frame that moves with its linear velocity (a Galilean
  // shift, exact: its acceleration changes by w x v, taken back below)
  o.V = l.root ? aba::v6<D>(x.vel.a, z3) : aba::zero6<D>();
  o.A0 = aba::v6<D>(z3, -gb);
  M3<D> Rl = R;
  V3<D> rl = l.rT;
  D py = x.pos.y;
  if (l.one) {
    if (l.jt == SIM_JOINT_PRISMATIC) {
      Rl = l.ETt;
      rl = axpy(rl, x.q, aba::mul(l.ETt, l.ax));
    } else {
      // rotation by q about the axis: 1 + sin q [a]x + (1 - cos q) [a]x^2
      D sn, cs;
      sincos(x.q, &sn, &cs);
      const D v = 1.0 - cs;
      const V3<D>& a = l.ax;
      const D aa = dot(a, a);
      M3<D> Q;
      Q.m[0] = 1.0 + v * (a.x * a.x - aa); Q.m[1] = v * a.x * a.y - sn * a.z; Q.m[2] = v * a.x * a.z + sn * a.y;
      Q.m[3] = v * a.x * a.y + sn * a.z; Q.m[4] = 1.0 + v * (a.y * a.y - aa); Q.m[5] = v * a.y * a.z - sn * a.x;
      Q.m[6] = v * a.x * a.z - sn * a.y; Q.m[7] = v * a.y * a.z + sn * a.x; Q.m[8] = 1.0 + v * (a.z * a.z - aa);
      Rl = aba::mul(l.ETt, Q);
    }
    if (l.p < 0) {
      py = rl.y;
      rl = z3;
    }
  }
  py = bc<0>(py);
  for (int d = 0; d <= tp.maxd; ++d) {
    if (l.dep == d) {
      if (l.one) {
        V6<D> Vp = aba::zero6<D>(), Ap = o.A0;
        if (l.p >= 0) {
          const D* q = g.X + l.p * kRec;
          const M3<D> Rp = ld9(q);
          const V3<D> d = aba::mul(Rp, rl);
          org = ld3(q + 9) + d;
          if constexpr (OWN) sh = d;
          R = aba::mul(Rp, Rl);
          Vp = ld6(q + 12);
          Ap = ld6(q + 18);
        } else {
          org = rl;
          R = Rl;
        }
        const V3<D> a = aba::mul(R, l.ax);
        o.S = l.jt == SIM_JOINT_PRISMATIC ? aba::v6<D>(z3, a) : aba::v6<D>(a, cross(org, a));
        const V6<D> vJ = x.qd * o.S;
        o.V = Vp + vJ;
        o.A0 = Ap + crm(o.V, vJ);
      }
      D* q = g.X + l.gl * kRec;
#pragma unroll
      for (int k = 0; k < 9; ++k) q[k] = R.m[k];
      st3(q + 9, org);
      st6(q + 12, o.V);
      st6(q + 18, o.A0);
    }
    sync();
  }
  // ---- contact rows: the sphere's centre and lowest point in the base
  // frame, the row's world direction there, the gap
  o.s = 1;
  const V3<D> e = aba::v3<D>(l.d == 1 ? 1.0 : 0.0, l.d == 0 ? 1.0 : 0.0, l.d == 2 ? 1.0 : 0.0);
  const V3<D> ey = aba::v3<D>(0.0, 1.0, 0.0);
  o.n = e;
  o.ny = ey;
  if (tp.free_root) {
    o.s = o.quat.x * o.quat.x + o.quat.y * o.quat.y + o.quat.z * o.quat.z + o.quat.w * o.quat.w;
    o.n = quat_rotate_T(o.quat, e);
    o.ny = quat_rotate_T(o.quat, ey);
  }
  o.cb = z3;
  o.phi = 1;
  if (l.k >= 0) {
    const D* q = g.X + l.cl * kRec;
    o.cb = ld3(q + 9) + aba::mul(ld9(q), l.cc);
    o.phi = py + dot(o.ny, o.cb) - l.rad;
  }
  o.act = l.k >= 0 && o.phi < 0;
  const unsigned long long live = __ballot(o.act);
  const unsigned row = (unsigned)(live >> (threadIdx.x & 48)) & 0x249;  // the normals' lanes
  o.na = __popc(row);
  unsigned long long w4 = live | live >> 32;
  w4 |= w4 >> 16;
  o.any = (int)((w4 & 1) | (w4 >> 2 & 2) | (w4 >> 4 & 4) | (w4 >> 6 & 8));
  o.pt = o.cb - l.rad * o.ny;
  o.Phi = o.act ? aba::v6<D>(cross(o.pt, o.n), o.n) : aba::zero6<D>();
  sync();
  // ---- articulated inertias and bias forces, leaves to root
  const V3<D> cw = org + aba::mul(R, l.com);
  o.I.m = l.m;
  o.I.mc = l.m * cw;
  const D c2 = dot(o.I.mc, cw);
  o.I.I = aba::cong(R, l.Ic) + aba::sy3<D>(c2 - o.I.mc.x * cw.x, c2 - o.I.mc.y * cw.y, c2 - o.I.mc.z * cw.z,
                                           -o.I.mc.x * cw.y, -o.I.mc.x * cw.z, -o.I.mc.y * cw.z);
  o.h = mul(o.I, o.V);
  // about the joint's own origin (OWN), or all of this about the base's
  Body I = o.I;
  V6<D> Sj = o.S;
  if constexpr (OWN) {
    const V3<D> c = aba::mul(R, l.com);
    I.mc = l.m * c;
    const D cc = dot(I.mc, c);
    I.I = aba::cong(R, l.Ic) + aba::sy3<D>(cc - I.mc.x * c.x, cc - I.mc.y * c.y, cc - I.mc.z * c.z, -I.mc.x * c.y,
                                          -I.mc.x * c.z, -I.mc.y * c.z);
    if (l.one) Sj = l.jt == SIM_JOINT_PRISMATIC ? o.S : aba::v6<D>(o.S.a, z3);
  }
  V6<D> F = OWN ? mul(I, down(org, o.A0)) + crf(down(org, o.V), mul(I, down(org, o.V))) : mul(I, o.A0) + crf(o.V, o.h);
  SySp<D> IA;
  IA.A = I.I;
  const V3<D>& mc = I.mc;
  IA.B.m[0] = 0;     IA.B.m[1] = -mc.z; IA.B.m[2] = mc.y;
  IA.B.m[3] = mc.z;  IA.B.m[4] = 0;     IA.B.m[5] = -mc.x;
  IA.B.m[6] = -mc.y; IA.B.m[7] = mc.x;  IA.B.m[8] = 0;
  IA.C = aba::sy3<D>(l.m, l.m, l.m, 0.0, 0.0, 0.0);
  D tau = u;
  if (tp.has_limits && l.one) {
    if (x.q > l.hi) tau = tau - l.lk * (x.q - l.hi) - l.ld * x.qd;
    else if (x.q < l.lo) tau = tau - l.lk * (x.q - l.lo) - l.ld * x.qd;
  }
  D uj = 0;
  o.Dinv = 0;
  for (int d = tp.maxd; d >= 0; --d) {
    if (l.dep == d) {
      for (int c = 0; c < l.ccn; ++c) {
        const D* q = g.X + (l.cf + c) * kRec;
        IA = IA + ld21(q);
        F = F + ld6(q + 21);
      }
      if (l.one) {
        o.U = aba::mul(IA, Sj);
        o.Dinv = 1.0 / dot(Sj, o.U);
        uj = tau - dot(Sj, F);
        if (l.p >= 0) {
          D* q = g.X + l.gl * kRec;
          st21(q, up(sh, aba::rank1_down(IA, o.U, o.Dinv)));
          st6(q + 21, up(sh, F + (uj * o.Dinv) * o.U));
        }
      }
    }
    sync();
  }
  if constexpr (OWN) o.U = up(org, o.U);
  // ---- accelerations, root to leaves
  V6<D> a0 = aba::zero6<D>();
  if (l.root) {
    D M[36], r[6];
    aba::sysp_dense(IA, M);
    D L[15], iv[6];
#pragma unroll
    for (int k = 5; k >= 0; --k) {
      iv[k] = 1.0 / M[7 * k];
#pragma unroll
      for (int i = 0; i < k; ++i) {
        const D f = M[6 * k + i] * iv[k];
        L[k * (k - 1) / 2 + i] = f;
#pragma unroll
        for (int j = 0; j <= i; ++j) M[6 * i + j] = fma(-f, M[6 * k + j], M[6 * i + j]);
      }
    }
#pragma unroll
    for (int k = 0; k < 15; ++k) g.rt[k] = L[k];
#pragma unroll
    for (int k = 0; k < 6; ++k) g.rt[15 + k] = iv[k];
    from6(-1.0 * F, r);
    root_up(g.rt, r);
    root_down(g.rt, r);
    a0 = to6(r);
  }
  o.qdd = down(tp, l, g, o, uj, a0, o.a);
  o.qdm = x.qd + dt * o.qdd;
  o.qdm6 = x.vel + dt * aba::v6<D>(a0.a, a0.l - cross(x.vel.a, x.vel.l));
  o.qd1 = o.qdm;
  o.qd16 = o.qdm6;
  o.y = 0;
  o.y6 = aba::zero6<D>();
  o.x = o.lamn = o.dinv = o.b = 0;
  if (REC) o.clo1 = o.chi1 = o.clo2 = o.chi2 = 0;
  if (!o.any) return;
  // ---- contact rows J, their eliminated form Z, and b = J qd_minus + ...
  if (l.one) {
    D* q = g.lk + l.gl * kLk;
    st6(q, o.S);
    st6(q + 6, o.Dinv * o.U);
    q[12] = o.Dinv;
    q[13] = o.qdm;
  }
  if (l.root) st6(g.rt + 21, o.qdm6);
  sync();
  const int dd = tp.dd;
  D zr[6] = {0, 0, 0, 0, 0, 0};
  const int i0 = walk_start(tp, l);
  if (l.k >= 0) {
    V6<D> p = aba::zero6<D>();
    D* const Jr = g.J + l.gl * dd;
    D* const Zr = g.Z + l.gl * dd;
    D bq = 0;
    for (int i = i0; i >= 0;) {
      const D* q = g.lk + i * kLk;
      const int mt = g.meta[i];
      const V6<D> Si = ld6(q);
      const D J = (mt & 1 ? 1.0 : o.s) * dot(Si, o.Phi);
      const D z = J - dot(Si, p);
      p = p + z * ld6(q + 6);
      bq = fma(J, q[13], bq);
      Jr[meta_slot(mt)] = J;
      Zr[meta_slot(mt)] = z;
      i = meta_par(mt);
    }
    if (tp.free_root) {
      D J[6];
      from6(aba::v6<D>(o.s * o.Phi.a, o.Phi.l), J);
      from6(p, zr);
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        bq = fma(J[k], g.rt[21 + k], bq);
        zr[k] = J[k] - zr[k];
        Jr[k] = J[k];
      }
      root_up(g.rt, zr);
#pragma unroll
      for (int k = 0; k < 6; ++k) Zr[k] = zr[k];
    }
    o.b = o.act ? (l.d == 0 ? bq + tp.beta / dt * o.phi : bq) : 0.0;
  }
  sync();
  // ---- A = Z^T D^-1 Z: the row's entries over the common parts of the paths
#pragma unroll
  for (int j = 0; j < kNR; ++j) o.A[j] = 0;
  if (l.k >= 0) {
    if (tp.free_root) {
#pragma unroll
      for (int k = 0; k < 6; ++k) zr[k] *= g.rt[15 + k];
#pragma unroll
      for (int j = 0; j < kNR; ++j) {
        if (j / 3 >= tp.nc) break;
        const D* Zj = g.Z + j * dd;
#pragma unroll
        for (int k = 0; k < 6; ++k) o.A[j] = fma(zr[k], Zj[k], o.A[j]);
      }
    }
    for (int i = i0; i >= 0;) {
      const int mt = g.meta[i], sl = meta_slot(mt);
      const D t = g.Z[l.gl * dd + sl] * g.lk[i * kLk + 12];
#pragma unroll
      for (int j = 0; j < kNR; ++j) {
        if (sl < l.nc4[j / 3]) o.A[j] = fma(t, g.Z[j * dd + sl], o.A[j]);
      }
      i = meta_par(mt);
    }
  }
  D diag = 0;
#pragma unroll
  for (int j = 0; j < kNR; ++j) {
    if (l.gl == j) {
      diag = o.A[j];
      o.A[j] = 0;
    }
  }
  const D dmax = rmax(diag);
  const bool keep = o.act && diag > 1e-12 * dmax;
  o.dinv = keep ? 1.0 / diag : 0.0;
  // ---- the normals alone, then all rows with the tangents boxed
  const D big = keep ? Big<D>::v : 0.0;
  D* const sw2 = g.X;
  D* const sw1 = g.X + kNR * (tp.niter + 1);
  const D x1 = sweeps<1, REC>(l, o, l.d == 0 ? o.dinv : 0.0, 0.0, l.d == 0 ? big : 0.0, tp.niter, sw1, kNC, o.clo1,
                              o.chi1);
  o.lamn = __shfl(x1, l.gl - l.d, kGrp);
  const D box = keep ? mu * o.lamn : 0.0;
  o.x = sweeps<3, REC>(l, o, o.dinv, l.d == 0 ? 0.0 : -box, l.d == 0 ? big : box, tp.niter, sw2, kNR, o.clo2, o.chi2);
  // ---- qd1 = qd_minus + M^-1 J^T x, from the eliminated rows: Z x, then
  // root to leaves.  The root's six entries are summed by lanes 0 to 5.
  D zx = 0, z0 = 0;
  unroll<kNR>([&](auto J) {
    if (o.any >> (J / 3) & 1) {
      const D xj = bc<J>(o.x);
      if (l.one && l.sph >> (J / 3) & 1) zx = fma(xj, g.Z[J * dd + l.slot], zx);
      if (tp.free_root && l.gl < 6) z0 = fma(xj, g.Z[J * dd + l.gl], z0);
    }
  });
  V6<D> ya = aba::zero6<D>();
  if (tp.free_root) {
    D r[6] = {bc<0>(z0), bc<1>(z0), bc<2>(z0), bc<3>(z0), bc<4>(z0), bc<5>(z0)};
    root_down(g.rt, r);
    o.y6 = to6(r);
    o.qd16 = o.qdm6 + o.y6;
  }
  if (REC) {
    // the exchange region holds the sweeps: the link's ancestors' responses
    // through the path instead (a few links), from the W region
    D* const ys = g.W;
    for (int d = 0; d <= tp.maxd; ++d) {
      if (l.dep == d && l.one) {
        V6<D> ap = tp.free_root ? o.y6 : aba::zero6<D>();
        for (int i = meta_par(g.meta[l.gl]); i >= 0; i = meta_par(g.meta[i])) ap = ap + ys[i] * ld6(g.lk + i * kLk);
        o.y = (zx - dot(o.U, ap)) * o.Dinv;
        ys[l.gl] = o.y;
      }
      sync();
    }
  } else {
    o.y = down(tp, l, g, o, zx, o.y6, ya);
  }
  o.qd1 = o.qdm + o.y;
}

__device__ __forceinline__ void integrate(const Lane& l, State& x, const Step& o, D dt) {
  if (l.one) {
    x.qd = o.qd1;
    x.q = x.q + dt * x.qd;
  }
  if (l.root) {
    x.vel = o.qd16;
    x.pos = axpy(x.pos, dt, quat_rotate(x.quat, x.vel.l));
    x.quat = aba::quat_step(x.quat, x.vel.a, dt);
  }
}

// One reversed solve: from xb (the adjoint of the result) and the recorded
// sweeps.  Row i's db_i = -y_bar_i / A_ii reaches the other lanes by
// broadcast; lane j collects column j of A_bar (the row read x_j at the end
// of the sweep for j < i, at its start for j > i, and y_i, the end value, for
// j = i where y_bar_i is not zero), b_bar of its own row, and the adjoints
// of its bounds.  A is symmetric: the lane's row serves as its column.
template <int ROWS>
__device__ __forceinline__ void sweeps_rev(const Lane& l, const Step& o, D xb, D dinv, int niter, const D* sw, int ld,
                                           unsigned long long clo, unsigned long long chi, D (&Ab)[kNR], D& bb,
                                           D& lob, D& hib) {
  const bool mine = l.k >= 0 && (ROWS == 3 || l.d == 0);
  const D* const my = sw + (ROWS == 3 ? l.gl : l.k);
  D xe = mine ? my[niter * ld] : 0.0;
  for (int it = niter - 1; it >= 0; --it) {
    const D xs = mine ? my[it * ld] : 0.0;
    const bool cl = clo >> it & 1, ch = chi >> it & 1;
    const D dv = cl || ch ? 0.0 : -dinv;
    D xl = 0;
    unroll<kNC>([&](auto Kr) {
      constexpr int K = kNC - 1 - Kr;
      if (o.any >> K & 1) {
        unroll<ROWS>([&](auto Rr) {
          constexpr int i = 3 * K + (ROWS - 1 - Rr);
          const bool own = l.gl == i;
          xl = own ? xb : xl;
          const D db = bc<i>(xb * dv);
          Ab[i] = fma(db, l.gl <= i ? xe : xs, Ab[i]);
          xb = fma(o.A[i], db, own ? 0.0 : xb);
        });
      }
    });
    bb = fma(xl, dv, bb);
    lob += cl ? xl : 0.0;
    hib += ch ? xl : 0.0;
    xe = xs;
  }
}

// The adjoint of the step at x, from what step<true> left in o and in the
// group's LDS (overwritten): xb in, the adjoint of (q1, qd1), and out, that of
// (q, qd); returns the control's adjoint, adds the friction coefficient's
// share of this lane to mub.
__device__ __forceinline__ D step_vjp(const WTopo& tp, const Lane& l, const Lds& g, const State& x, D dt, D mu,
                                      State& xb, D& mub, const Step& o) {
  const V3<D> z3 = aba::zero3<D>();
  const int dd = tp.dd;
  // ---- integrator
  D qb = xb.q, gl = xb.qd + dt * xb.q;
  V6<D> g6 = xb.vel;
  V3<D> pb = xb.pos;
  Q4<D> quatb = {0, 0, 0, 0};
  if (l.root) {
    quatb = aba::quat_step_adj(x.quat, o.qd16.a, dt, xb.quat, g6.a);
    const Q4<D> t = quat_rot_grad(x.quat, dt * pb, o.qd16.l);
    quatb = {quatb.x + t.x, quatb.y + t.y, quatb.z + t.z, quatb.w + t.w};
    g6.l = g6.l + quat_rotate_T(x.quat, dt * pb);
  }
  D qdmb = gl;
  V6<D> qdmb6 = g6;
  if (o.any) {
    const D bdt = tp.beta / dt;
    const int i0 = walk_start(tp, l);
    if (l.one) g.lk[l.gl * kLk + 14] = gl;
    if (l.root) st6(g.rt + 27, g6);
    sync();
    // ---- W = M^-1 J^T, one column per row lane (W[dof][row]); x_bar = W^T g
    D xbar = 0;
    const int off = tp.free_root ? 5 : 0;
    if (l.gl < kNR) {
      D r[6] = {0, 0, 0, 0, 0, 0};
      if (tp.free_root) {
        if (l.k >= 0) {
#pragma unroll
          for (int k = 0; k < 6; ++k) r[k] = g.Z[l.gl * dd + k];
          root_down(g.rt, r);
        }
#pragma unroll
        for (int k = 0; k < 6; ++k) {
          g.W[k * kNR + l.gl] = r[k];
          xbar = fma(r[k], g.rt[27 + k], xbar);
        }
      }
      const V6<D> ar = to6(r);
      for (int i = tp.free_root; i < tp.n; ++i) {
        const D* q = g.lk + i * kLk;
        const V6<D> Ud = ld6(q + 6);
        const int mt = g.meta[i];
        D w = -dot(Ud, ar);
        for (int j = meta_par(mt); j >= 0; j = meta_par(g.meta[j]))
          w = fma(-dot(Ud, ld6(g.lk + j * kLk)), g.W[(j + off) * kNR + l.gl], w);
        if (l.k >= 0 && tp.sph[i] >> l.k & 1) w = fma(q[12], g.Z[l.gl * dd + meta_slot(mt)], w);
        g.W[(i + off) * kNR + l.gl] = w;
        xbar = fma(w, q[14], xbar);
      }
    }
    // ---- the two solves, last first
    D Ab[kNR];
#pragma unroll
    for (int j = 0; j < kNR; ++j) Ab[j] = 0;
    D bb = 0, lob = 0, hib = 0;
    sweeps_rev<3>(l, o, xbar, o.dinv, tp.niter, g.X, kNR, o.clo2, o.chi2, Ab, bb, lob, hib);
    const D gb = l.d == 0 || l.gl >= kNR ? 0.0 : hib - lob;
    mub = fma(o.lamn, gb, mub);
    const D g1 = __shfl(gb, l.gl + 1, kGrp), g2 = __shfl(gb, l.gl + 2, kGrp);
    const D xn = l.d == 0 && l.k >= 0 ? mu * (g1 + g2) : 0.0;
    D t0 = 0, t1 = 0;
    sweeps_rev<1>(l, o, xn, l.d == 0 ? o.dinv : 0.0, tp.niter, g.X + kNR * (tp.niter + 1), kNC, o.clo1, o.chi1, Ab,
                  bb, t0, t1);
    sync();  // the sweeps are done with
    // ---- h = M^-1 g, and with it up the tree the composite inertias
    Body Ic = o.I;
    D h = gl;
    V6<D> h6 = g6;
    {
      for (int d = tp.maxd; d >= 0; --d) {
        if (l.dep == d) {
          V6<D> p = aba::zero6<D>();
          for (int c = 0; c < l.ccn; ++c) {
            const D* q = g.X + (l.cf + c) * kRec;
            p = p + ld6(q);
            Ic.m += q[6];
            Ic.mc = Ic.mc + ld3(q + 7);
            Ic.I = Ic.I + aba::sy3<D>(q[10], q[11], q[12], q[13], q[14], q[15]);
          }
          if (l.one) {
            h = h - dot(o.S, p);
            if (l.p >= 0) {
              D* q = g.X + l.gl * kRec;
              st6(q, p + (h * o.Dinv) * o.U);
              q[6] = Ic.m;
              st3(q + 7, Ic.mc);
              q[10] = Ic.I.xx; q[11] = Ic.I.yy; q[12] = Ic.I.zz; q[13] = Ic.I.xy; q[14] = Ic.I.xz; q[15] = Ic.I.yz;
            }
          } else {
            h6 = h6 - p;
          }
        }
        sync();
      }
      V6<D> a0 = aba::zero6<D>();
      if (l.root) {
        D r[6];
        from6(h6, r);
        root_up(g.rt, r);
        root_down(g.rt, r);
        a0 = to6(r);
      }
      h6 = a0;
      V6<D> a;
      h = down(tp, l, g, o, h, a0, a);
    }
    // ---- C = A_bar + A_bar^T, y and h by degree of freedom, Ic S by link
    D* const C = g.X;
    D* const Y = C + kNR * kNR;
    D* const H = Y + tp.nv;
    D* const FS = H + tp.nv;
    D* const N = FS + 6 * kGrp;
    if (l.gl < kNR) {
#pragma unroll
      for (int j = 0; j < kNR; ++j) C[j * kNR + l.gl] = Ab[j];
    }
    if (l.one) {
      Y[l.dof] = o.y;
      H[l.dof] = h;
      st6(FS + 6 * l.gl, mul(Ic, o.S));
    }
    if (l.root) {
      st6(Y, o.y6);
      st6(H, h6);
    }
    sync();
    if (l.gl < kNR) {
#pragma unroll
      for (int j = 0; j < kNR; ++j) Ab[j] += C[l.gl * kNR + j];
    }
    sync();
    if (l.gl < kNR) {
#pragma unroll
      for (int j = 0; j < kNR; ++j) C[j * kNR + l.gl] = Ab[j];
    }
    // ---- b = J qd_minus + ...: qd_minus_bar += J^T b_bar (the root's six
    // entries in lanes 0 to 5)
    D r0 = 0;
    unroll<kNR>([&](auto J) {
      if (o.any >> (J / 3) & 1) {
        const D bj = bc<J>(bb);
        if (l.one && l.sph >> (J / 3) & 1) qdmb = fma(bj, g.J[J * dd + l.slot], qdmb);
        if (tp.free_root && l.gl < 6) r0 = fma(bj, g.J[J * dd + l.gl], r0);
      }
    });
    if (tp.free_root) {
      const D r[6] = {bc<0>(r0), bc<1>(r0), bc<2>(r0), bc<3>(r0), bc<4>(r0), bc<5>(r0)};
      qdmb6 = qdmb6 + to6(r);
    }
    sync();
    // ---- J_bar = C W^T + b_bar qd_minus^T + x h^T along the row's path, and
    // through J = S . Phi to the wrench Phi and the joint subspaces: a change
    // of q_m turns every S_k beyond it into S_k + S_m x S_k
    Q4<D> qg = {0, 0, 0, 0};
    D pyb = 0;
    if (l.k >= 0) {
      D* const Jr = g.J + l.gl * dd;
      auto jbar = [&](int dof, D qdm) {
        D v = fma(bb, qdm, o.x * H[dof]);
#pragma unroll
        for (int j = 0; j < kNR; ++j) v = fma(Ab[j], g.W[dof * kNR + j], v);
        return o.act ? v : 0.0;
      };
      V6<D> Pb = aba::zero6<D>();
      D sb = 0;
      for (int i = i0; i >= 0;) {
        const int mt = g.meta[i];
        const D* q = g.lk + i * kLk;
        const D v = jbar(i + off, q[13]);
        if (!(mt & 1)) sb = fma(v, Jr[meta_slot(mt)], sb);
        Pb = Pb + ((mt & 1 ? 1.0 : o.s) * v) * ld6(q);
        Jr[meta_slot(mt)] = v;
        i = meta_par(mt);
      }
      if (tp.free_root) {
        D v[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
          v[k] = jbar(k, g.rt[21 + k]);
          if (k < 3) {
            sb = fma(v[k], Jr[k], sb);
            v[k] *= o.s;
          }
        }
        Pb = Pb + to6(v);
      }
      const V3<D> ptb = cross(o.n, Pb.a);
      const V3<D> nb = cross(Pb.a, o.pt) + Pb.l;
      const D phib = l.d == 0 && o.act ? bdt * bb : 0.0;
      const V3<D> cbb = axpy(ptb, phib, o.ny);
      const V3<D> nyb = axpy(-l.rad * ptb, phib, o.cb);
      if (tp.free_root) {
        const V3<D> e = aba::v3<D>(l.d == 1 ? 1.0 : 0.0, l.d == 0 ? 1.0 : 0.0, l.d == 2 ? 1.0 : 0.0);
        const Q4<D> a = quat_rot_grad(o.quat, e, nb), b = quat_rot_grad(o.quat, aba::v3<D>(0.0, 1.0, 0.0), nyb);
        const D f = 2 * sb / o.s;
        qg = {a.x + b.x + f * o.quat.x, a.y + b.y + f * o.quat.y, a.z + b.z + f * o.quat.z,
              a.w + b.w + f * o.quat.w};
        if (!o.act) qg = {0, 0, 0, 0};
        pyb = phib;
      }
      const V6<D> Psi = aba::v6<D>(cross(o.cb, cbb), cbb);
      V6<D> run = aba::zero6<D>();
      for (int i = i0; i >= 0;) {
        const int mt = g.meta[i];
        const V6<D> Si = ld6(g.lk + i * kLk);
        const D v = Jr[meta_slot(mt)];
        Jr[meta_slot(mt)] = o.act ? dot(Si, crf(run, o.Phi) + Psi) : 0.0;
        run = run + ((mt & 1 ? 1.0 : o.s) * v) * Si;
        i = meta_par(mt);
      }
    }
    if (tp.free_root) {
      const D s0 = rsum(qg.x), s1 = rsum(qg.y), s2 = rsum(qg.z), s3 = rsum(qg.w), s4 = rsum(pyb);
      if (l.root) {
        quatb = {quatb.x + s0, quatb.y + s1, quatb.z + s2, quatb.w + s3};
        pb.y += s4;
      }
    }
    // ---- the adjoint of M is -N / 2, N = W C W^T + h y^T + y h^T, kept for
    // pairs on one path (N[dof][slot of the ancestor])
    auto nrow = [&](int a, D (&T)[kNR]) {
#pragma unroll
      for (int j = 0; j < kNR; ++j) T[j] = 0;
#pragma unroll
      for (int r = 0; r < kNR; ++r) {
        const D w = g.W[a * kNR + r];
#pragma unroll
        for (int j = 0; j < kNR; ++j) T[j] = fma(w, C[r * kNR + j], T[j]);
      }
    };
    auto nent = [&](const D (&T)[kNR], D y, D hh, int c) {
      D v = fma(y, H[c], hh * Y[c]);
#pragma unroll
      for (int j = 0; j < kNR; ++j) v = fma(T[j], g.W[c * kNR + j], v);
      return v;
    };
    if (l.one) {
      D T[kNR];
      nrow(l.dof, T);
      for (int i = l.gl; i >= 0;) {
        const int mt = g.meta[i];
        N[l.dof * dd + meta_slot(mt)] = nent(T, o.y, h, i + off);
        i = meta_par(mt);
      }
      if (tp.free_root)
        for (int k = 0; k < 6; ++k) N[l.dof * dd + k] = nent(T, o.y, h, k);
    }
    if (tp.free_root && l.gl < 6) {
      D T[kNR];
      nrow(l.gl, T);
      const D y = Y[l.gl], hh = H[l.gl];
      for (int k = 0; k < 6; ++k)
        if (k <= l.gl) N[l.gl * dd + k] = nent(T, y, hh, k);
    }
    sync();
    // ---- q_bar += sum over strict ancestors a of (S_k x S_a) . (Ic_k X_a +
    // Y_a), X_a = sum over strict ancestors c of S_c N_ac, Y_a = sum over
    // the subtree's links j of Ic_j S_j N_ja
    if (l.one) {
      const int first = meta_par(g.meta[l.gl]);
      auto share = [&](int da, int sa, const V6<D>& Sa) {
        V6<D> X = aba::zero6<D>();
        if (tp.free_root) {
          D r[6];
#pragma unroll
          for (int c = 0; c < 6; ++c) r[c] = c <= da ? N[da * dd + c] : N[c * dd + sa];
          X = to6(r);
        }
        for (int c = first; c >= 0;) {
          const int mc_ = g.meta[c], sc = meta_slot(mc_);
          const D v = sc <= sa ? N[da * dd + sc] : N[(c + off) * dd + sa];
          X = X + v * ld6(g.lk + c * kLk);
          c = meta_par(mc_);
        }
        V6<D> G = mul(Ic, X);
        for (int m = l.sub; m; m &= m - 1) {
          const int j = __ffs(m) - 1;
          G = G + N[(j + off) * dd + sa] * ld6(FS + 6 * j);
        }
        qb += dot(crm(o.S, Sa), G);
      };
      if (tp.free_root)
        for (int k = 0; k < 6; ++k)
          share(k, k,
                aba::v6<D>(aba::v3<D>(k == 0 ? 1.0 : 0.0, k == 1 ? 1.0 : 0.0, k == 2 ? 1.0 : 0.0),
                           aba::v3<D>(k == 3 ? 1.0 : 0.0, k == 4 ? 1.0 : 0.0, k == 5 ? 1.0 : 0.0)));
      for (int i = first; i >= 0;) {
        const int mt = g.meta[i];
        share(i + off, meta_slot(mt), ld6(g.lk + i * kLk));
        i = meta_par(mt);
      }
      // the rows' shares through J and the contact points
#pragma unroll
      for (int j = 0; j < kNR; ++j)
        if (l.sph >> (j / 3) & 1) qb += g.J[j * dd + l.slot];
    }
    sync();
  }
  // ---- the smooth step, qd_minus = qd + dt FD(q, qd, u): w = M^-1 (dt
  // qd_minus_bar), then the adjoint of <w, ID(q, qd, qdd)> at fixed qdd
  D w = dt * qdmb;
  V6<D> w6 = dt * qdmb6, Bv;
  minv(tp, l, g, o, w, w6, Bv);
  const V6<D> A = o.a + o.A0;
  V6<D> Gb = mul(o.I, Bv), F = mul(o.I, A) + crf(o.V, o.h);
  for (int d = tp.maxd; d >= 0; --d) {
    if (l.dep == d) {
      for (int c = 0; c < l.ccn; ++c) {
        const D* q = g.X + (l.cf + c) * kRec;
        Gb = Gb + ld6(q);
        F = F + ld6(q + 6);
      }
      if (l.p >= 0) {
        D* q = g.X + l.gl * kRec;
        st6(q, Gb);
        st6(q + 6, F);
      }
    }
    sync();
  }
  const V6<D> vJ = x.qd * o.S;
  V6<D> vb = crmT(Bv, o.h) - mul(o.I, crm(o.V, Bv));
  if (l.one) vb = vb - crmT(vJ, Gb);
  for (int d = tp.maxd; d >= 0; --d) {
    if (l.dep == d) {
      for (int c = 0; c < l.ccn; ++c) vb = vb + ld6(g.X + (l.cf + c) * kRec);
      if (l.p >= 0) st6(g.X + l.gl * kRec, vb);
    }
    sync();
  }
  if (l.one) {
    // the subtree turns with q: its parent's B, A and V enter it turned back
    const V6<D> Bp = Bv - w * o.S, Ap = A - o.qdd * o.S - crm(o.V, vJ), Vp = o.V - vJ;
    const D qE = -dot(o.S, crf(Bp, F) + crf(Ap, Gb) + crf(Vp, vb));
    const D qdE = dot(o.S, crmT(o.V, Gb) + vb);
    xb.q = qb - qE;
    xb.qd = qdmb - qdE;
    if (tp.has_limits && (x.q > l.hi || x.q < l.lo)) {
      xb.q -= l.lk * w;
      xb.qd -= l.ld * w;
    }
  }
  if (l.root) {
    const Q4<D> t = quat_rot_grad(x.quat, aba::v3<D>(tp.g[0], tp.g[1], tp.g[2]), Gb.l);
    xb.pos = pb;
    xb.quat = {quatb.x + t.x, quatb.y + t.y, quatb.z + t.z, quatb.w + t.w};
    xb.vel = aba::v6<D>(qdmb6.a - vb.a - cross(x.vel.l, Gb.l), qdmb6.l - cross(Gb.l, x.vel.a));
  }
  return w;
}

}  // namespace wave

#endif  // __HIPCC__

}  // namespace aba_contact
