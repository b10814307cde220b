// World positions of one point per system from its joint coordinates, and
// the adjoint (the loss side of Sec. 3, Eq. diff_u: dPhi/dx^T enters the
// adjoint recursion).
//
// A point sees only its link's path to the root: the links' poses are
// composed down the path, R_i = R_p E_T^T R_j(q), p_i = p_p + R_p r (R_j a
// rotation: 1 + sin q [a]x + (1 - cos q) [a]x^2 revolute, R(quat) spherical;
// r = r_T + q E_T^T a prismatic; a free root is R(quat), p itself).
//
// One wavefront per system, one lane per path link (root first): the lanes
// load their links and form R_j at once; the chain of products then runs in
// uniform registers, link after link, each lane keeping what the adjoint of
// its own joint needs, and the joint adjoints are formed by all lanes at
// once.  What bounds it is that chain: about 60 dependent operations a link
// each way.  2048 chains of 5 to 50 links: 20 us forward and 35 us with the
// adjoint's, where a tree level at a time took about 30 launches a level,
// 45 ms in all.  A scan over the lanes would be shorter, but rounds in
// another order: the seeds of ill-conditioned chains amplify that (up to
// 3e-5 in the gradient over 50 steps in FP32).  So the products keep the torch
// expressions' order; their sums of three are fused multiply-adds in index
// order, where a library's product may round otherwise.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>

#include "../../include/abadj.h"
#include "aba_lane.h"
#include "abadj_internal.h"

namespace {

using aba::M3;
using aba::Q4;
using aba::V3;
constexpr int kWaveLanes = 64;
constexpr int kSysPerBlock = 4;

template <typename S>
struct FkArgs {
  int nsys, len;        // systems, entries of a path
  const int32_t* path;  // [nsys][len]: link, root first, -1 past the end
  const int32_t* jtype;  // [n_links]
  const int64_t* qidx;   // [n_links]
  const S* ETt;          // [n_links][9]: joint frame -> parent
  const S* rT;           // [n_links][3]
  const S* ax;           // [n_links][3]
  const S* pts;          // [nsys][3]
  const S* q;
  S* x;                  // forward: [nsys][3]
  const S* xbar;         // adjoint: [nsys][3]
  S* gq;                 // adjoint: entries of the paths' joints are written
};

template <typename S>
__device__ __forceinline__ S dot3(S a0, S b0, S a1, S b1, S a2, S b2) {
  return fma(a2, b2, fma(a1, b1, a0 * b0));
}
template <typename S>
__device__ __forceinline__ M3<S> mm(const M3<S>& A, const M3<S>& B) {  // A B
  M3<S> C;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      C.m[3 * i + j] = dot3(A.m[3 * i], B.m[j], A.m[3 * i + 1], B.m[3 + j], A.m[3 * i + 2], B.m[6 + j]);
  return C;
}
template <typename S>
__device__ __forceinline__ V3<S> mv(const M3<S>& A, const V3<S>& v) {
  return aba::v3<S>(dot3(A.m[0], v.x, A.m[1], v.y, A.m[2], v.z), dot3(A.m[3], v.x, A.m[4], v.y, A.m[5], v.z),
                    dot3(A.m[6], v.x, A.m[7], v.y, A.m[8], v.z));
}
template <typename S>
__device__ __forceinline__ M3<S> eye() {
  M3<S> m;
#pragma unroll
  for (int k = 0; k < 9; ++k) m.m[k] = k % 4 == 0 ? S(1) : S(0);
  return m;
}
// the value of lane j in every lane
__device__ __forceinline__ float lane_of(float x, int j) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), j));
}
__device__ __forceinline__ double lane_of(double x, int j) {
  const long long v = __double_as_longlong(x);
  const unsigned lo = __builtin_amdgcn_readlane((int)v, j), hi = __builtin_amdgcn_readlane((int)(v >> 32), j);
  return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}
template <typename S>
__device__ __forceinline__ V3<S> lane_of(const V3<S>& v, int j) {
  return aba::v3<S>(lane_of(v.x, j), lane_of(v.y, j), lane_of(v.z, j));
}
template <typename S>
__device__ __forceinline__ M3<S> lane_of(const M3<S>& m, int j) {
  M3<S> r;
#pragma unroll
  for (int k = 0; k < 9; ++k) r.m[k] = lane_of(m.m[k], j);
  return r;
}

// A path link: its transform, and after compose() its parent's pose.
template <typename S>
struct Link {
  int jt;  // -1: past the end of the path
  int64_t qi;
  M3<S> ET, K, K2, J;  // joint frame -> parent; [a]x and its square; R_j
  V3<S> a, r;
  S s, c;
  Q4<S> quat;
  M3<S> A1;  // R_p E_T^T
  M3<S> Rp;
};

template <typename S>
__device__ __forceinline__ M3<S> quat_matrix(const Q4<S>& q) {
  M3<S> R;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const V3<S> e = aba::v3<S>(S(j == 0), S(j == 1), S(j == 2));
    const V3<S> c = aba::quat_rotate(q, e);
    R.m[j] = c.x;
    R.m[3 + j] = c.y;
    R.m[6 + j] = c.z;
  }
  return R;
}
__device__ __forceinline__ float sin_(float x) { return sinf(x); }
__device__ __forceinline__ float cos_(float x) { return cosf(x); }
__device__ __forceinline__ double sin_(double x) { return sin(x); }
__device__ __forceinline__ double cos_(double x) { return cos(x); }

template <typename S>
__device__ __forceinline__ Link<S> load_link(const FkArgs<S>& A, int sys, int lane) {
#pragma clang fp contract(off)
  Link<S> l;
  const int i = lane < A.len ? A.path[(size_t)sys * A.len + lane] : -1;
  l.jt = i < 0 ? -1 : A.jtype[i];
  l.J = l.ET = eye<S>();
  l.a = l.r = aba::zero3<S>();
  l.s = l.c = S(0);
  l.quat = {S(0), S(0), S(0), S(1)};
  l.qi = 0;
  l.K = l.K2 = l.A1 = l.Rp = eye<S>();
  if (i < 0) return l;
  l.qi = A.qidx[i];
#pragma unroll
  for (int k = 0; k < 9; ++k) l.ET.m[k] = A.ETt[9 * (size_t)i + k];
  l.a = aba::v3<S>(A.ax[3 * (size_t)i], A.ax[3 * (size_t)i + 1], A.ax[3 * (size_t)i + 2]);
  l.r = aba::v3<S>(A.rT[3 * (size_t)i], A.rT[3 * (size_t)i + 1], A.rT[3 * (size_t)i + 2]);
  auto at = [&](int k) { return A.q[l.qi + k]; };
  if (l.jt == SIM_JOINT_FREE) {  // its own pose, whatever E_T and r_T say
    l.quat = {at(3), at(4), at(5), at(6)};
    l.ET = eye<S>();
    l.r = aba::v3<S>(at(0), at(1), at(2));
    l.J = quat_matrix(l.quat);
  } else if (l.jt == SIM_JOINT_SPHERICAL) {
    l.quat = {at(0), at(1), at(2), at(3)};
    l.J = quat_matrix(l.quat);
  } else if (l.jt == SIM_JOINT_PRISMATIC) {
    const S q = at(0);
    const V3<S> t = mv(l.ET, aba::v3<S>(q * l.a.x, q * l.a.y, q * l.a.z));
    l.r = aba::v3<S>(l.r.x + t.x, l.r.y + t.y, l.r.z + t.z);
  } else {
    l.s = sin_(at(0));
    l.c = cos_(at(0));
    const V3<S>& a = l.a;
    l.K.m[0] = 0;    l.K.m[1] = -a.z; l.K.m[2] = a.y;
    l.K.m[3] = a.z;  l.K.m[4] = 0;    l.K.m[5] = -a.x;
    l.K.m[6] = -a.y; l.K.m[7] = a.x;  l.K.m[8] = 0;
    l.K2 = mm(l.K, l.K);
    const S v = S(1) - l.c;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const S t = S(k % 4 == 0) + l.s * l.K.m[k];
      l.J.m[k] = t + v * l.K2.m[k];
    }
  }
  return l;
}

// Composes the path's poses; each lane keeps its parent's.
template <typename S>
__device__ __forceinline__ void compose(Link<S>& l, int lane, int len, M3<S>& R, V3<S>& p) {
#pragma clang fp contract(off)
  R = eye<S>();
  p = aba::zero3<S>();
  for (int j = 0; j < len; ++j) {
    if (__builtin_amdgcn_readlane(l.jt, j) < 0) break;
    const V3<S> t = mv(R, lane_of(l.r, j));
    const M3<S> A1 = mm(R, lane_of(l.ET, j));
    if (lane == j) {
      l.Rp = R;
      l.A1 = A1;
    }
    p = aba::v3<S>(p.x + t.x, p.y + t.y, p.z + t.z);
    R = mm(A1, lane_of(l.J, j));
  }
}

template <typename S>
__global__ __launch_bounds__(kWaveLanes* kSysPerBlock) void k_link_points(FkArgs<S> A) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x % kWaveLanes;
  const int sys = blockIdx.x * kSysPerBlock + threadIdx.x / kWaveLanes;
  if (sys >= A.nsys) return;  // whole wavefronts
  Link<S> l = load_link(A, sys, lane);
  M3<S> R;
  V3<S> p;
  compose(l, lane, A.len, R, p);
  if (lane == 0) {
    const S* c = A.pts + 3 * (size_t)sys;
    const V3<S> t = mv(R, aba::v3<S>(c[0], c[1], c[2]));
    S* o = A.x + 3 * (size_t)sys;
    o[0] = p.x + t.x;
    o[1] = p.y + t.y;
    o[2] = p.z + t.z;
  }
}

// The adjoints of the poses back along the path, gR and gp; lane j keeps
// gR at its own link, from which its joint's adjoint follows.
template <typename S>
__global__ __launch_bounds__(kWaveLanes* kSysPerBlock) void k_link_points_adj(FkArgs<S> A) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x % kWaveLanes;
  const int sys = blockIdx.x * kSysPerBlock + threadIdx.x / kWaveLanes;
  if (sys >= A.nsys) return;
  Link<S> l = load_link(A, sys, lane);
  M3<S> R, gR, own = eye<S>();
  V3<S> p;
  compose(l, lane, A.len, R, p);
  const S* c = A.pts + 3 * (size_t)sys;
  const S* xb = A.xbar + 3 * (size_t)sys;
  const V3<S> g = aba::v3<S>(xb[0], xb[1], xb[2]);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    gR.m[k] = g.x * c[k];
    gR.m[3 + k] = g.y * c[k];
    gR.m[6 + k] = g.z * c[k];
  }
  for (int j = A.len - 1; j >= 0; --j) {
    if (__builtin_amdgcn_readlane(l.jt, j) < 0) continue;
    if (lane == j) own = gR;
    const M3<S> J = lane_of(l.J, j), E = lane_of(l.ET, j);
    const V3<S> r = lane_of(l.r, j);
    const M3<S> gA = mm(gR, aba::transpose(J)), gP = mm(gA, aba::transpose(E));
    const S rr[3] = {r.x, r.y, r.z}, gg[3] = {g.x, g.y, g.z};
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int k = 0; k < 3; ++k) gR.m[3 * i + k] = gP.m[3 * i + k] + gg[i] * rr[k];
  }
  if (l.jt < 0) return;
  S* o = A.gq + l.qi;
  if (l.jt == SIM_JOINT_PRISMATIC) {
    const V3<S> ge = mv(aba::transpose(l.ET), mv(aba::transpose(l.Rp), g));
    o[0] = ge.x * l.a.x + ge.y * l.a.y + ge.z * l.a.z;
    return;
  }
  const M3<S> gJ = mm(aba::transpose(l.A1), own);
  if (l.jt == SIM_JOINT_REVOLUTE) {
    S gs = 0, gc = 0;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      gs += gJ.m[k] * l.K.m[k];
      gc += gJ.m[k] * l.K2.m[k];
    }
    o[0] = gs * l.c + gc * l.s;
    return;
  }
  // R(quat): the gradient of sum_k gJ e_k^T R e_k
  Q4<S> t = {S(0), S(0), S(0), S(0)};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const V3<S> e = aba::v3<S>(S(k == 0), S(k == 1), S(k == 2));
    const Q4<S> u = aba::quat_rot_grad(l.quat, aba::v3<S>(gJ.m[k], gJ.m[3 + k], gJ.m[6 + k]), e);
    t = {t.x + u.x, t.y + u.y, t.z + u.z, t.w + u.w};
  }
  if (l.jt == SIM_JOINT_FREE) {
    o[0] = g.x;
    o[1] = g.y;
    o[2] = g.z;
    o += 3;
  }
  o[0] = t.x;
  o[1] = t.y;
  o[2] = t.z;
  o[3] = t.w;
}

template <typename S>
hipError_t launch(const FkArgs<S>& a, bool adjoint, hipStream_t st) {
  const dim3 grid((a.nsys + kSysPerBlock - 1) / kSysPerBlock), block(kWaveLanes * kSysPerBlock);
  if (adjoint) hipLaunchKernelGGL((k_link_points_adj<S>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((k_link_points<S>), grid, block, 0, st, a);
  return hipGetLastError();
}

template <typename S>
int run(const char* who, int nsys, int len, const int32_t* path, const int32_t* jtype, const int64_t* qidx,
        const void* ETt, const void* rT, const void* ax, const void* pts, const void* q, void* x, const void* xbar,
        void* gq, void* stream) {
  const FkArgs<S> a{nsys, len, path, jtype, qidx, (const S*)ETt, (const S*)rT, (const S*)ax, (const S*)pts,
                    (const S*)q, (S*)x, (const S*)xbar, (S*)gq};
  const hipError_t e = launch(a, xbar != nullptr, (hipStream_t)stream);
  if (e != hipSuccess)
    return aba::report_error(SIM_ERR_HIP, std::string(who) + ": launch failed: " + hipGetErrorString(e));
  return SIM_OK;
}

int points(const char* who, int dtype, int nsys, int len, const int32_t* path, const int32_t* jtype,
           const int64_t* qidx, const void* ETt, const void* rT, const void* ax, const void* pts, const void* q,
           void* x, const void* xbar, void* gq, void* stream) {
  aba::clear_error();
  if (dtype != SIM_F32 && dtype != SIM_F64)
    return aba::report_error(SIM_ERR_UNSUPPORTED_DTYPE, std::string(who) + ": dtype must be SIM_F32 or SIM_F64");
  if (nsys < 0 || len < 1 || len > SIM_MAX_LINKS)
    return aba::report_error(SIM_ERR_INVALID_ARG, std::string(who) + ": need n_sys >= 0 and 1 <= len <= " +
                                                      std::to_string(SIM_MAX_LINKS));
  if (nsys == 0) return SIM_OK;
  if (!path || !jtype || !qidx || !ETt || !rT || !ax || !pts || !q || !(xbar ? gq : x))
    return aba::report_error(SIM_ERR_INVALID_ARG, std::string(who) + ": null array argument");
  return dtype == SIM_F64
             ? run<double>(who, nsys, len, path, jtype, qidx, ETt, rT, ax, pts, q, x, xbar, gq, stream)
             : run<float>(who, nsys, len, path, jtype, qidx, ETt, rT, ax, pts, q, x, xbar, gq, stream);
}

}  // namespace

extern "C" {

int sim_link_points(int dtype, int n_sys, int len, const int32_t* path, const int32_t* jtype, const int64_t* qidx,
                    const void* ETt, const void* rT, const void* ax, const void* pts, const void* q, void* x,
                    void* stream) {
  return points("sim_link_points", dtype, n_sys, len, path, jtype, qidx, ETt, rT, ax, pts, q, x, nullptr, nullptr,
                stream);
}

int sim_link_points_adjoint(int dtype, int n_sys, int len, const int32_t* path, const int32_t* jtype,
                            const int64_t* qidx, const void* ETt, const void* rT, const void* ax, const void* pts,
                            const void* q, const void* xbar, void* gq, void* stream) {
  if (n_sys > 0 && !xbar) {
    aba::clear_error();
    return aba::report_error(SIM_ERR_INVALID_ARG, "sim_link_points_adjoint: null array argument");
  }
  return points("sim_link_points_adjoint", dtype, n_sys, len, path, jtype, qidx, ETt, rT, ax, pts, q, nullptr, xbar,
                gq, stream);
}

}  // extern "C"
