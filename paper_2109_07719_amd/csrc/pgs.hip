// Contact solver for gfx950: projected Gauss-Seidel (PGS) on a batch of
// independent mixed linear complementarity problems, and its adjoint.
//
// Problem (Sec. 4.1 "Collision resolution", Eq. mlcp; App. C): find x with
//   a = A x + b,  lo <= x <= hi,  a_i >= 0 where x_i = lo_i,
//   a_i <= 0 where x_i = hi_i,  a_i = 0 in between,
// by niter sweeps from a start x0; each sweep sets the rows in order,
//   y_i = -(b_i + sum_{j != i} A_ij x_j) / A_ii,  x_i = min(max(y_i, lo_i), hi_i).
// The adjoint reverses the sweeps (App. C: the reverse solver mirrors the
// forward one with the adjoint of every operation) from the vector stored
// at the start of every sweep: the clamp sends x_bar_i to the active bound
// or to y_bar_i, then b_bar_i, A_bar_i. and x_bar_j (j != i) follow from
// y_i, and x_bar_i is reset.
//
// Layout on the GPU: four lanes (a quad) per problem, sixteen problems per
// wavefront; lane g holds the columns j = 4 c + g of A (and of A_bar) and the
// vectors' entries j.  A row's sum is the lanes' partial sums joined by two
// quad permutations; the row is then finished by every lane with its own
// entry c and kept by the one that owns it, so that no per-row quantity is
// held four times.  A kernel is compiled for 4, 8, 12 and 16 rows: row and
// column loops are unrolled and every operand has a fixed register, A_bar's
// too; the up to three rows past n are zero rows, which leave everything as it
// is, and no branch separates one row's instructions from the next's.  The
// sweep vectors go to the workspace as [niter + 1][n][batch].  Problems are
// independent: no barriers.  Problems of up to four rows that fill the chip
// take a lane each (launch says from where on): G lanes per problem, 4 or 1.
//
// What bounds it: the instructions of a row, the GS order being a serial chain
// of n niter rows.  With one lane per problem 32768 problems were 512
// wavefronts, half a SIMD's worth each, every lane reading rows of A of its
// own, with A and A_bar (288 registers of 12 rows) past the register file.
// 32768 problems x 12 rows x 30 sweeps, FP32: solve 59 -> 29 us, adjoint 138
// -> 71 us, and in FP64 71 -> 41 and 2033 -> 96; 64 problems 35 -> 17 and 93 ->
// 33; 16 rows, 32768 problems, 92 -> 39 and 445 -> 113; 4 rows 18 -> 11 and 29
// -> 18; 200000 problems of 4 rows 32 -> 29 and 60 -> 48.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>

#include "../../include/abadj.h"
#include "abadj_internal.h"

namespace {

constexpr int kBlock = 64;  // sixteen problems; blocks of 128 and 256 are no faster at any batch

template <typename S>
struct PgsArgs {
  int batch, n, niter;
  const S* A;    // [batch][n][n]
  const S* b;    // [batch][n]
  const S* lo;
  const S* hi;
  const S* x0;
  S* x;          // solve: result [batch][n]
  S* ws;         // nullable (solve) / required (adjoint): [niter + 1][n][batch]
  const S* xbar; // adjoint: seed [batch][n]
  S* Abar;       // adjoint outputs
  S* bbar;
  S* lobar;
  S* hibar;
  S* x0bar;
};

// x of another lane of the quad (CTRL: a quad permutation)
template <int CTRL>
__device__ __forceinline__ float quad(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double quad(double x) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true));
}
// the sum over a problem's G lanes
template <int G, typename S>
__device__ __forceinline__ S lane_sum(S x) {
  if constexpr (G == 1) return x;
  x += quad<0xB1>(x);  // [1, 0, 3, 2]
  return x + quad<0x4E>(x);  // [2, 3, 0, 1]
}

// x / d by a reciprocal taken once, rounded as the division would be.  FP32: by
// way of FP64.  FP64: the product and its remainder, which rounds to the
// quotient (Markstein's theorem); the last instruction is the division's own,
// for zeros and infinities.
template <typename S>
struct Reciprocal;
template <>
struct Reciprocal<float> {
  double r;
  __device__ __forceinline__ void set(float d) { r = 1.0 / double(d); }
  __device__ __forceinline__ float times(float x) const { return float(double(x) * r); }
};
template <>
struct Reciprocal<double> {
  double d, r;
  __device__ __forceinline__ void set(double d_) {
    d = d_;
    r = fabs(d) < 0x1p-1022 ? copysign(0x1.fffffffffffffp1023, d) : 1.0 / d;  // (no infinite product)
  }
  __device__ __forceinline__ double times(double x) const {
    const double q = x * r;
    return __builtin_amdgcn_div_fixup(fma(fma(-d, q, x), r, q), d, x);
  }
};

// A problem's columns and bounds on one of its G lanes
template <typename S, int N, int G>
struct Problem {
  static constexpr int C = N / G;
  int n, g;
  size_t p;
  S A[N][C];                  // off-diagonal; zero on the diagonal and past n
  S b[C], lo[C], hi[C];
  Reciprocal<S> inv[C];       // of A_jj

  __device__ __forceinline__ size_t at(int c) const { return p * n + G * c + g; }
  __device__ __forceinline__ bool has(int c) const { return G * c + g < n; }
  __device__ __forceinline__ bool owns(int i) const { return g == i % G && i < n; }
  __device__ __forceinline__ void load(S (&v)[C], const S* src, size_t first, size_t stride) const {
#pragma unroll
    for (int c = 0; c < C; ++c) v[c] = has(c) ? src[first + (G * c + g) * stride] : S(0);
  }
  __device__ __forceinline__ void store(const S (&v)[C], S* dst, size_t first, size_t stride) const {
#pragma unroll
    for (int c = 0; c < C; ++c)
      if (has(c)) dst[first + (G * c + g) * stride] = v[c];
  }
  __device__ __forceinline__ Problem(const PgsArgs<S>& P, size_t p_, int g_) : n(P.n), g(g_), p(p_) {
    S d[C];
#pragma unroll
    for (int c = 0; c < C; ++c) d[c] = S(1);
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const S v = (i < n && has(c)) ? P.A[(p * n + i) * n + G * c + g] : S(0);
        const bool diag = i == G * c + g;
        A[i][c] = diag ? S(0) : v;
        if (diag && i < n) d[c] = v;
      }
    load(b, P.b, p * n, 1);
    load(lo, P.lo, p * n, 1);
    load(hi, P.hi, p * n, 1);
#pragma unroll
    for (int c = 0; c < C; ++c) inv[c].set(d[c]);
  }
  // x / A_jj of the lane's entry c
  __device__ __forceinline__ S over(S x, int c) const { return inv[c].times(x); }
  // y of row i, on the lane that owns it, from the vector x
  __device__ __forceinline__ S row(int i, const S (&x)[C]) const {
    S d = S(0);
#pragma unroll
    for (int c = 0; c < C; ++c) d = fma(A[i][c], c == i / G && owns(i) ? S(0) : x[c], d);  // x_i may be infinite
    d = lane_sum<G>(d);
    return over(-(b[i / G] + d), i / G);
  }
};

template <typename S, int N, int G>
__global__ __launch_bounds__(kBlock) void k_pgs_solve(PgsArgs<S> P) {
  constexpr int C = N / G;
  const size_t p = ((size_t)blockIdx.x * kBlock + threadIdx.x) / G;
  if (p >= (size_t)P.batch) return;  // whole problems
  const size_t B = (size_t)P.batch, n = (size_t)P.n;
  const Problem<S, N, G> m(P, p, threadIdx.x % G);
  S x[C];
  m.load(x, P.x0, p * n, 1);
  for (int t = 0; t < P.niter; ++t) {
    if (P.ws) m.store(x, P.ws + p, t * n * B, B);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int c = i / G;
      const S y = m.row(i, x);
      const S v = (y < m.lo[c]) ? m.lo[c] : ((y > m.hi[c]) ? m.hi[c] : y);
      x[c] = m.owns(i) ? v : x[c];
    }
  }
  m.store(x, P.x, p * n, 1);
  if (P.ws) m.store(x, P.ws + p, P.niter * n * B, B);
}

template <typename S, int N, int G>
__global__ __launch_bounds__(kBlock) void k_pgs_adjoint(PgsArgs<S> P) {
  constexpr int C = N / G;
  const size_t p = ((size_t)blockIdx.x * kBlock + threadIdx.x) / G;
  if (p >= (size_t)P.batch) return;  // whole problems
  const size_t B = (size_t)P.batch, n = (size_t)P.n;
  const Problem<S, N, G> m(P, p, threadIdx.x % G);
  // A_bar sums in FP64, from x widened once a sweep: its error does not grow
  // with the sweeps (relative error against FP64, 20 sweeps, 16 rows, FP32:
  // 1.15e-7 with FP32 sums, 6.9e-8 so, 7.2e-8 with the sums begun at the first
  // sweep)
  double Ab[N][C], xd[C];
  S Ad[C], xb[C], bb[C], lb[C], hb[C], x[C], xs[C], nx[C];
  m.load(xb, P.xbar, p * n, 1);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    Ad[c] = bb[c] = lb[c] = hb[c] = x[c] = nx[c] = S(0);
#pragma unroll
    for (int i = 0; i < N; ++i) Ab[i][c] = 0.0;
  }
  // x: before row i of sweep t it holds the sweep's end for j < i and its
  // start, xs, for j > i; so at the sweep's first row it holds the start, the
  // end of the sweep before
  if (P.niter > 0) {
    m.load(x, P.ws + p, P.niter * n * B, B);
    m.load(nx, P.ws + p, (P.niter - 1) * n * B, B);
  }
#pragma unroll
  for (int c = 0; c < C; ++c) xd[c] = double(x[c]);
  for (int t = P.niter - 1; t >= 0; --t) {
#pragma unroll
    for (int c = 0; c < C; ++c) xs[c] = nx[c];
    if (t > 0) m.load(nx, P.ws + p, (t - 1) * n * B, B);
#pragma unroll
    for (int i = N - 1; i >= 0; --i) {
      const int c = i / G;
      const bool own = m.owns(i);
      const S y = m.row(i, x);
      const S t0 = own ? xb[c] : S(0);
      const bool below = y < m.lo[c], above = !below && y > m.hi[c];
      lb[c] += below ? t0 : S(0);
      hb[c] += above ? t0 : S(0);
      const S own_db = -m.over(below || above ? S(0) : t0, c);
      bb[c] += own_db;
      Ad[c] += own ? own_db * y : S(0);
      S db = own_db;
      if constexpr (G == 4)
        db = i % 4 == 0 ? quad<0x00>(own_db) : i % 4 == 1 ? quad<0x55>(own_db)
           : i % 4 == 2 ? quad<0xAA>(own_db) : quad<0xFF>(own_db);
#pragma unroll
      for (int k = 0; k < C; ++k) {
        Ab[i][k] = fma(double(db), xd[k], Ab[i][k]);
        xb[k] = fma(db, m.A[i][k], xb[k]);
      }
      xb[c] = own ? S(0) : xb[c];
      x[c] = own ? xs[c] : x[c];
      xd[c] = own ? double(xs[c]) : xd[c];
    }
  }
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (i < P.n) {
#pragma unroll
      for (int c = 0; c < C; ++c)
        if (m.has(c)) P.Abar[(p * n + i) * n + G * c + m.g] = i == G * c + m.g ? Ad[c] : S(Ab[i][c]);
    }
  m.store(bb, P.bbar, p * n, 1);
  m.store(lb, P.lobar, p * n, 1);
  m.store(hb, P.hibar, p * n, 1);
  m.store(xb, P.x0bar, p * n, 1);
}

int pgs_fail(int code, const std::string& msg) { return aba::report_error(code, msg); }

// the sweep vectors [niter + 1][n][batch]; past 12 rows callers provide
// [niter][n][batch] more, which the kernels leave alone
size_t pgs_ws_bytes(int dtype, int batch, int n, int niter) {
  const size_t rows = (size_t)(niter + 1) + (n > 12 ? (size_t)niter : 0);
  return rows * (size_t)n * (size_t)batch * (dtype == SIM_F64 ? sizeof(double) : sizeof(float));
}

int pgs_check(const char* who, int dtype, int batch, int n, int niter) {
  if (dtype != SIM_F32 && dtype != SIM_F64)
    return pgs_fail(SIM_ERR_UNSUPPORTED_DTYPE, std::string(who) + ": dtype must be SIM_F32 or SIM_F64");
  if (batch < 0 || niter < 0 || n < 1 || n > SIM_PGS_MAX_ROWS)
    return pgs_fail(SIM_ERR_INVALID_ARG, std::string(who) + ": need batch >= 0, niter >= 0 and 1 <= n <= " +
                                             std::to_string(SIM_PGS_MAX_ROWS));
  return SIM_OK;
}

// SIMDs of the current device
int simd_count() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 1024;
  return 4 * cus;
}

// one kernel per row bucket (4, 8, 12, 16 with four lanes, 2 and 4 with one)
template <typename S, int N, int G>
void launch_n(const PgsArgs<S>& a, hipStream_t st, bool adjoint) {
  const dim3 grid((unsigned)(((size_t)a.batch * G + kBlock - 1) / kBlock));
  if (adjoint) hipLaunchKernelGGL((k_pgs_adjoint<S, N, G>), grid, dim3(kBlock), 0, st, a);
  else hipLaunchKernelGGL((k_pgs_solve<S, N, G>), grid, dim3(kBlock), 0, st, a);
}
template <typename S>
hipError_t launch(const PgsArgs<S>& a, hipStream_t st, bool adjoint) {
  if (a.batch == 0) return hipSuccess;
  // One lane per problem for one or two rows (32768 problems of two, FP32, four
  // lanes / one: solve 10 / 8 us, adjoint 19 / 9; 64 of them 8 / 8 and 12 / 8), and
  // for up to four where four lanes would take more than one wavefront per SIMD
  // (4 rows, 16384 problems 10 / 10 and 14 / 16, 24576 10 / 11 and 19 / 17, 200000
  // 35 / 29 and 89 / 49; FP64 24576 16 / 13 and 27 / 20, 200000 70 / 46 and 133 /
  // 80).  From five rows up A and A_bar no longer fit one lane's registers.
  if (a.n <= 2) launch_n<S, 2, 1>(a, st, adjoint);
  else if (a.n <= 4 && (size_t)a.batch * 4 > (size_t)kBlock * simd_count()) launch_n<S, 4, 1>(a, st, adjoint);
  else if (a.n <= 4) launch_n<S, 4, 4>(a, st, adjoint);
  else if (a.n <= 8) launch_n<S, 8, 4>(a, st, adjoint);
  else if (a.n <= 12) launch_n<S, 12, 4>(a, st, adjoint);
  else launch_n<S, 16, 4>(a, st, adjoint);
  return hipGetLastError();
}

}  // namespace

extern "C" {

int sim_pgs_workspace_bytes(int dtype, int batch, int n, int niter, size_t* bytes) {
  aba::clear_error();
  if (!bytes) return pgs_fail(SIM_ERR_INVALID_ARG, "sim_pgs_workspace_bytes: null argument");
  const int rc = pgs_check("sim_pgs_workspace_bytes", dtype, batch, n, niter);
  if (rc) return rc;
  *bytes = pgs_ws_bytes(dtype, batch, n, niter);
  return SIM_OK;
}

int sim_pgs_solve(int dtype, int batch, int n, int niter, const void* A, const void* b, const void* lo,
                  const void* hi, const void* x0, void* x, void* workspace, size_t workspace_bytes, void* stream) {
  aba::clear_error();
  int rc = pgs_check("sim_pgs_solve", dtype, batch, n, niter);
  if (rc) return rc;
  if (batch > 0 && (!A || !b || !lo || !hi || !x0 || !x))
    return pgs_fail(SIM_ERR_INVALID_ARG, "sim_pgs_solve: null array argument");
  if (workspace && workspace_bytes < pgs_ws_bytes(dtype, batch, n, niter))
    return pgs_fail(SIM_ERR_WORKSPACE_TOO_SMALL, "sim_pgs_solve: workspace of " + std::to_string(workspace_bytes) +
                                                     " bytes, need " +
                                                     std::to_string(pgs_ws_bytes(dtype, batch, n, niter)));
  hipError_t e;
  if (dtype == SIM_F64) {
    PgsArgs<double> a{batch, n, niter, (const double*)A, (const double*)b, (const double*)lo, (const double*)hi,
                      (const double*)x0, (double*)x, (double*)workspace, nullptr, nullptr, nullptr, nullptr,
                      nullptr, nullptr};
    e = launch<double>(a, (hipStream_t)stream, false);
  } else {
    PgsArgs<float> a{batch, n, niter, (const float*)A, (const float*)b, (const float*)lo, (const float*)hi,
                     (const float*)x0, (float*)x, (float*)workspace, nullptr, nullptr, nullptr, nullptr,
                     nullptr, nullptr};
    e = launch<float>(a, (hipStream_t)stream, false);
  }
  if (e != hipSuccess) return pgs_fail(SIM_ERR_HIP, std::string("sim_pgs_solve: launch failed: ") + hipGetErrorString(e));
  return SIM_OK;
}

int sim_pgs_adjoint(int dtype, int batch, int n, int niter, const void* A, const void* b, const void* lo,
                    const void* hi, const void* xbar, void* workspace, size_t workspace_bytes, void* Abar,
                    void* bbar, void* lobar, void* hibar, void* x0bar, void* stream) {
  aba::clear_error();
  int rc = pgs_check("sim_pgs_adjoint", dtype, batch, n, niter);
  if (rc) return rc;
  if (batch > 0 && (!A || !b || !lo || !hi || !xbar || !workspace || !Abar || !bbar || !lobar || !hibar || !x0bar))
    return pgs_fail(SIM_ERR_INVALID_ARG, "sim_pgs_adjoint: null array argument");
  if (workspace_bytes < pgs_ws_bytes(dtype, batch, n, niter))
    return pgs_fail(SIM_ERR_WORKSPACE_TOO_SMALL, "sim_pgs_adjoint: workspace of " +
                                                     std::to_string(workspace_bytes) + " bytes, need " +
                                                     std::to_string(pgs_ws_bytes(dtype, batch, n, niter)));
  hipError_t e;
  if (dtype == SIM_F64) {
    PgsArgs<double> a{batch, n, niter, (const double*)A, (const double*)b, (const double*)lo, (const double*)hi,
                      nullptr, nullptr, (double*)workspace, (const double*)xbar, (double*)Abar, (double*)bbar,
                      (double*)lobar, (double*)hibar, (double*)x0bar};
    e = launch<double>(a, (hipStream_t)stream, true);
  } else {
    PgsArgs<float> a{batch, n, niter, (const float*)A, (const float*)b, (const float*)lo, (const float*)hi,
                     nullptr, nullptr, (float*)workspace, (const float*)xbar, (float*)Abar, (float*)bbar,
                     (float*)lobar, (float*)hibar, (float*)x0bar};
    e = launch<float>(a, (hipStream_t)stream, true);
  }
  if (e != hipSuccess)
    return pgs_fail(SIM_ERR_HIP, std::string("sim_pgs_adjoint: launch failed: ") + hipGetErrorString(e));
  return SIM_OK;
}

}  // extern "C"
