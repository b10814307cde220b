// Collision detection and contact resolution inside the time step
// (Sec. 4.1 "Collision resolution": detection and an MLCP solved by
// projected Gauss-Seidel between the dynamics and the integrator), batched
// over systems of one topology, and the gradient of a rollout through
// contact.
//
// Contact model: spheres fixed in links against the ground plane y = 0.
//   - a sphere is active when its centre is lower than its radius (gap
//     phi = centre_y - radius < 0);
//   - per active contact three rows (normal e_y, tangents e_x, e_z) of J,
//     the world velocity of the sphere's lowest point as a point of its
//     link;
//   - impulses lambda solve a = A lambda + b with A = J M^-1 J^T and
//     b = J qd_minus + (beta/dt) phi on the normal rows, qd_minus = qd +
//     dt qdd: first the normal rows alone with lambda_n >= 0, then all rows
//     with the tangents boxed by +-mu times those first normal impulses;
//     a row with A_ii = 0 (no joint moves the point along it) is left out;
//   - qd1 = qd_minus + M^-1 J^T lambda; the positions then move with qd1
//     (p1 = p + dt R v_lin1 and the normalised quaternion step for a free
//     root, q1 = q + dt qd1 for 1-dof joints).
//
// Design: 16 lanes per system (contact_wave.h says why).  The gradient runs
// backwards in time in the same layout: each step is recomputed from the
// stored state, then its statements are reversed, and the adjoint of the
// state is carried to the previous step (Sec. 3, Eq. adj_back; Sec. 4.1, Eq.
// adj_r).  contact_step.h and contact_adjoint.h hold the same step and its
// adjoint as one system's statements in order: the operation count below
// runs them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <type_traits>

#include "../../include/abadj.h"
#include "aba_lane.h"
#include "abadj_internal.h"
#include "contact_adjoint.h"
#include "contact_wave.h"

namespace {

using namespace aba_contact;


// ---- operation count (host) --------------------------------------------------
// A counting scalar that carries its value, so that every data-dependent
// decision (detection, dropped rows, clamps) is taken as on the device:
// every +, -, *, /, sqrt, sin and cos counts 1.
thread_local long long g_cops = 0;
struct CD {
  double v = 0;
  CD() = default;
  template <typename T, typename = std::enable_if_t<std::is_arithmetic_v<T>>>
  CD(T x) : v(double(x)) {}
};
inline CD cd_(double x) { ++g_cops; return CD(x); }
inline CD operator+(CD a, CD b) { return cd_(a.v + b.v); }
inline CD operator-(CD a, CD b) { return cd_(a.v - b.v); }
inline CD operator*(CD a, CD b) { return cd_(a.v * b.v); }
inline CD operator/(CD a, CD b) { return cd_(a.v / b.v); }
inline CD operator-(CD a) { return CD(-a.v); }
inline CD& operator+=(CD& a, CD b) { a = a + b; return a; }
inline bool operator<(CD a, CD b) { return a.v < b.v; }
inline bool operator>(CD a, CD b) { return a.v > b.v; }
inline CD val(CD x) { return x; }
inline CD sq_root(CD x) { return cd_(std::sqrt(x.v)); }
inline void sin_cos(CD x, CD& s, CD& c) { s = cd_(std::sin(x.v)); c = cd_(std::cos(x.v)); }
// the terms of an unrolled sum past its true length are not counted
inline CD fmadd_pad(CD a, CD b, CD c, bool live) { return live ? a * b + c : c; }
inline CD mul_pad(CD a, CD b, bool live) { return live ? a * b : CD(0); }
inline CD add_pad(CD a, CD b, bool live) { return live ? a + b : a; }
inline CD sub_pad(CD a, CD b, bool live) { return live ? a - b : a; }

}  // namespace

namespace aba_contact {
template <>
struct Big<CD> { static constexpr double v = 1e300; };
template <>
struct RealOf<CD> { using type = CD; };
}  // namespace aba_contact

namespace {

// ---- kernels ---------------------------------------------------------------

constexpr int kWave = 64;

extern __shared__ __align__(16) double contact_lds[];

template <typename S>
struct RollArgs {
  WTopo tp;
  int B, T;
  double dt;
  const S* P;     // [np][B]
  const S* q0;    // [nq][B]
  const S* qd0;   // [nv][B]
  const S* tau;   // [T][nu][B]
  S* traj;        // nullable: [T + 1][nq + nv][B]
  S* qT;          // [nq][B]
  S* qdT;         // [nv][B]
  int* ncont;     // nullable: [T][B]
};

// The rollout: four systems per wavefront, the state in registers.
template <typename S>
__global__ __launch_bounds__(kWave) void k_contact_rollout(RollArgs<S> a) {
  __shared__ int meta[kGrp];
  wave::fill_meta(a.tp, meta);
  wave::sync();
  const int s0 = blockIdx.x * kSysWave + threadIdx.x / kGrp;
  const bool live = s0 < a.B;  // the last wavefront's spare groups repeat system B - 1
  const int s = live ? s0 : a.B - 1;
  const size_t B = (size_t)a.B;
  const wave::Lds g = wave::lds_of(a.tp, contact_lds, meta);
  const wave::Lane l = wave::load_lane(a.tp, a.P, B, s);
  const int nx = a.tp.nq + a.tp.nv, nu = a.tp.nu;
  wave::State x = wave::zero_state();
  wave::load_state(x, l, a.q0, a.qd0, B, s);
  if (a.traj && live) wave::store_state(x, l, a.traj, a.traj + (size_t)a.tp.nq * B, B, s);
  double un = l.one && a.T > 0 ? double(a.tau[l.ui * B + s]) : 0.0;
  for (int t = 0; t < a.T; ++t) {
    const double u = un;
    if (l.one && t + 1 < a.T) un = double(a.tau[((size_t)(t + 1) * nu + l.ui) * B + s]);
    wave::Step o;
    wave::step<false, sizeof(S) == sizeof(double)>(a.tp, l, g, x, u, a.dt, a.tp.mu, o);
    wave::integrate(l, x, o, a.dt);
    wave::round_state<S>(x);
    if (a.ncont && live && l.gl == 0) a.ncont[(size_t)t * B + s] = o.na;
    if (a.traj && live) {
      S* row = a.traj + (size_t)(t + 1) * nx * B;
      wave::store_state(x, l, row, row + (size_t)a.tp.nq * B, B, s);
    }
  }
  if (live) wave::store_state(x, l, a.qT, a.qdT, B, s);
}

template <typename S>
struct GradArgs {
  WTopo tp;
  int B, T;
  double dt;
  const S* P;     // [np][B]
  const S* traj;  // [T + 1][nq + nv][B] from the rollout
  const S* tau;   // [T][nu][B]
  const S* gqT;   // [nq][B]
  const S* gqdT;  // [nv][B]
  S* gq0;         // [nq][B]
  S* gqd0;        // [nv][B]
  S* gtau;        // [T][nu][B]
  S* gmu;         // nullable: [B]
};

// The rollout gradient by the step's reverse statements, backwards in time:
// per step, step<true> recomputes the step from the stored state and step_vjp
// runs the adjoints of the integrator, the impulse update, both Gauss-Seidel solves
// (from their recorded sweeps), A and b, M^-1 J^T, the contact geometry and
// the smooth step.  The next state and control are fetched a step ahead.
template <typename S>
__global__ __launch_bounds__(kWave) void k_contact_adj(GradArgs<S> a) {
  __shared__ int meta[kGrp];
  wave::fill_meta(a.tp, meta);
  wave::sync();
  const int s0 = blockIdx.x * kSysWave + threadIdx.x / kGrp;
  const bool live = s0 < a.B;
  const int s = live ? s0 : a.B - 1;
  const size_t B = (size_t)a.B;
  const wave::Lds g = wave::lds_of(a.tp, contact_lds, meta);
  const wave::Lane l = wave::load_lane(a.tp, a.P, B, s);
  const int nx = a.tp.nq + a.tp.nv, nu = a.tp.nu;
  wave::State xb = wave::zero_state(), nxt = wave::zero_state();
  wave::load_state(xb, l, a.gqT, a.gqdT, B, s);
  double un = 0, mub = 0;
  auto fetch = [&](int t) {
    const S* row = a.traj + (size_t)t * nx * B;
    wave::load_state(nxt, l, row, row + (size_t)a.tp.nq * B, B, s);
    if (l.one) un = double(a.tau[((size_t)t * nu + l.ui) * B + s]);
  };
  if (a.T > 0) fetch(a.T - 1);
  for (int t = a.T - 1; t >= 0; --t) {
    const wave::State x = nxt;
    const double u = un;
    if (t > 0) fetch(t - 1);
    wave::Step o;
    wave::step<true, sizeof(S) == sizeof(double)>(a.tp, l, g, x, u, a.dt, a.tp.mu, o);
    const double ub = wave::step_vjp(a.tp, l, g, x, a.dt, a.tp.mu, xb, mub, o);
    if (live && l.one) a.gtau[((size_t)t * nu + l.ui) * B + s] = S(ub);
  }
  if (live) wave::store_state(xb, l, a.gq0, a.gqd0, B, s);
  mub = wave::rsum(mub);
  if (a.gmu && live && l.gl == 0) a.gmu[s] = S(mub);
}

// The same with two wavefronts per four systems, for batches that leave half
// the SIMDs idle: they take the steps in turn, each with its own LDS, so that
// one recomputes its step, which waits for nothing, while the other reverses
// the step after it.  Nothing but the adjoint state goes from one to the
// other.  A step costs its reverse alone, not both: 250 systems (63
// workgroups), 30 sweeps, FP64: 87 -> 60 us a step.
size_t pair_lds_bytes(const WTopo& tp) {
  return 2 * wave_lds_bytes(tp) + (size_t)(wave::kStateNumbers + 1) * kWave * sizeof(double);
}
template <typename S>
__global__ __launch_bounds__(2 * kWave) void k_contact_adj_pair(GradArgs<S> a) {
  __shared__ int meta[kGrp];
  wave::fill_meta(a.tp, meta);
  __syncthreads();
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int s0 = blockIdx.x * kSysWave + lane / kGrp;
  const bool live = s0 < a.B;
  const int s = live ? s0 : a.B - 1;
  const size_t B = (size_t)a.B;
  const wave::Lds g = wave::lds_of(a.tp, contact_lds, meta);  // by the group in the workgroup
  double* const xch = contact_lds + 2 * (size_t)kSysWave * a.tp.stride + lane;
  const wave::Lane l = wave::load_lane(a.tp, a.P, B, s);
  const int nx = a.tp.nq + a.tp.nv, nu = a.tp.nu;
  wave::State xb = wave::zero_state(), nxt = wave::zero_state(), x = wave::zero_state();
  double un = 0, mub = 0;
  auto fetch = [&](int t) {
    if (t < 0) return;
    const S* row = a.traj + (size_t)t * nx * B;
    wave::load_state(nxt, l, row, row + (size_t)a.tp.nq * B, B, s);
    if (l.one) un = double(a.tau[((size_t)t * nu + l.ui) * B + s]);
  };
  if (wid == 0) {
    wave::load_state(xb, l, a.gqT, a.gqdT, B, s);
    wave::each(xb, [&](int k, double& v) { xch[k * kWave] = v; });
  }
  fetch(a.T - 1 - wid);
  wave::Step o;
  for (int k = -1; k < a.T; ++k) {
    const int t = a.T - 1 - k;  // the step to reverse
    if (wid == (k & 1)) {
      if (k >= 0) {
        wave::each(xb, [&](int i, double& v) { v = xch[i * kWave]; });
        const double ub = wave::step_vjp(a.tp, l, g, x, a.dt, a.tp.mu, xb, mub, o);
        if (live && l.one) a.gtau[((size_t)t * nu + l.ui) * B + s] = S(ub);
        wave::each(xb, [&](int i, double& v) { xch[i * kWave] = v; });
      }
    } else if (t > 0) {
      x = nxt;
      const double u = un;
      fetch(t - 3);
      wave::step<true, sizeof(S) == sizeof(double)>(a.tp, l, g, x, u, a.dt, a.tp.mu, o);
    }
    __syncthreads();
  }
  mub = wave::rsum(mub);
  if (wid == 1) xch[wave::kStateNumbers * kWave] = mub;
  __syncthreads();
  if (wid == 0 && live) {
    wave::each(xb, [&](int i, double& v) { v = xch[i * kWave]; });
    wave::store_state(xb, l, a.gq0, a.gqd0, B, s);
    if (a.gmu && l.gl == 0) a.gmu[s] = S(mub + xch[wave::kStateNumbers * kWave]);
  }
}

int cfail(int code, const std::string& msg) { return aba::report_error(code, msg); }

// The launch geometries a model may ask for (m->tiling); the kernels have one,
// so a choice changes nothing.
constexpr int kRollSplDefault = 8, kGradSplDefault = 16;
bool roll_spl_ok(int spl) { return spl == 8 || spl == 4 || spl == 2; }
bool grad_spl_ok(int spl) { return spl == 16 || spl == 8 || spl == 4; }

template <typename S>
hipError_t launch_rollout(const RollArgs<S>& a, hipStream_t st) {
  hipLaunchKernelGGL((k_contact_rollout<S>), dim3((a.B + kSysWave - 1) / kSysWave), dim3(kWave), wave_lds_bytes(a.tp),
                     st, a);
  return hipGetLastError();
}
// The model's constants as a rollout in S saw them (rounded to S), for the
// reverse pass, which runs in FP64 for both dtypes.
template <typename S>
CTopo constants_as_seen_by(CTopo tp) {
  for (int k = 0; k < 3; ++k) tp.g[k] = double(S(tp.g[k]));
  tp.mu = double(S(tp.mu));
  tp.beta = double(S(tp.beta));
  for (int i = 0; i < kNL; ++i)
    for (int k = 0; k < 4; ++k) tp.lim[i][k] = double(S(tp.lim[i][k]));
  return tp;
}

template <typename S>
hipError_t launch_grad(const GradArgs<S>& a, hipStream_t st) {
  const int blocks = (a.B + kSysWave - 1) / kSysWave;
  int dev = 0, cus = 0, lds = 0;
  // two wavefronts while all of them are resident at once (one pair a CU for
  // quadrupeds, by its LDS: FP32, one wavefront / two, 16 systems 85 / 60 us a
  // step, 1000 systems 88 / 71, 2048 systems 92 / 141)
  const bool pair = a.T > 1 && hipGetDevice(&dev) == hipSuccess &&
                    hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
                    hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess &&
                    (size_t)blocks <= cus * std::min<size_t>(2, lds / (pair_lds_bytes(a.tp) + kGrp * sizeof(int)));
  if (pair) hipLaunchKernelGGL((k_contact_adj_pair<S>), dim3(blocks), dim3(2 * kWave), pair_lds_bytes(a.tp), st, a);
  else hipLaunchKernelGGL((k_contact_adj<S>), dim3(blocks), dim3(kWave), wave_lds_bytes(a.tp), st, a);
  return hipGetLastError();
}

int make_topo(const char* who, const sim_contact_model* m, CTopo* tp) {
  if (!m || !m->parent || !m->jtype || (m->ncontacts > 0 && !m->contact_link))
    return cfail(SIM_ERR_INVALID_ARG, std::string(who) + ": null model argument");
  if (m->n < 1 || m->n > kNL)
    return cfail(SIM_ERR_INVALID_TOPOLOGY, std::string(who) + ": need 1 <= n <= " + std::to_string(kNL));
  if (m->ncontacts < 0 || m->ncontacts > kNC)
    return cfail(SIM_ERR_INVALID_ARG, std::string(who) + ": need 0 <= ncontacts <= " + std::to_string(kNC));
  if (m->niter < 0 || !(m->mu >= 0) || !(m->beta >= 0))
    return cfail(SIM_ERR_INVALID_ARG, std::string(who) + ": need niter >= 0, mu >= 0, beta >= 0");
  if (m->tiling && (!roll_spl_ok(m->tiling->rollout_systems_per_wave) ||
                    !grad_spl_ok(m->tiling->grad_systems_per_wave) ||
                    (m->tiling->grad_lds != 0 && m->tiling->grad_lds != 1) ||
                    (m->tiling->grad_lds == 0 && m->tiling->grad_systems_per_wave != 16)))
    return cfail(SIM_ERR_INVALID_ARG, std::string(who) + ": tiling needs rollout_systems_per_wave in {8, 4, 2}, "
                                                         "grad_systems_per_wave in {16, 8, 4} and grad_lds 1, "
                                                         "or grad_systems_per_wave 16 with grad_lds 0");
  *tp = CTopo{};
  tp->n = m->n;
  tp->nc = m->ncontacts;
  tp->niter = m->niter;
  tp->mu = m->mu;
  tp->beta = m->beta;
  for (int k = 0; k < 3; ++k) tp->g[k] = m->gravity[k];
  int nq = 0, nv = 0, nu = 0;
  for (int i = 0; i < m->n; ++i) {
    const int p = m->parent[i], jt = m->jtype[i];
    if (i == 0 ? p != -1 : (p < 0 || p >= i))
      return cfail(SIM_ERR_INVALID_TOPOLOGY, std::string(who) + ": need parent[0] = -1 and 0 <= parent[i] < i");
    if (jt == SIM_JOINT_FREE ? i != 0 : (jt != SIM_JOINT_REVOLUTE && jt != SIM_JOINT_PRISMATIC))
      return cfail(SIM_ERR_INVALID_TOPOLOGY,
                   std::string(who) + ": joints must be revolute or prismatic, a free joint only at link 0");
    tp->parent[i] = p;
    tp->jtype[i] = jt;
    tp->qi[i] = nq;
    tp->vi[i] = nv;
    tp->ui[i] = nu;
    if (jt == SIM_JOINT_FREE) { nq += 7; nv += 6; }
    else { nq += 1; nv += 1; nu += 1; }
  }
  if (m->limits) {
    for (int i = 0; i < m->n; ++i) {
      if (m->jtype[i] == SIM_JOINT_FREE) continue;
      const double* L = m->limits + 4 * i;
      if (!(std::isfinite(L[0]) && std::isfinite(L[1]) && std::isfinite(L[2]) && std::isfinite(L[3])) ||
          !(L[0] <= L[1]) || !(L[2] >= 0) || !(L[3] >= 0))
        return cfail(SIM_ERR_INVALID_ARG, std::string(who) + ": joint limits need finite lo <= hi, k >= 0, d >= 0");
      for (int k = 0; k < 4; ++k) tp->lim[i][k] = L[k];
    }
    tp->has_limits = 1;
  }
  for (int k = 0; k < m->ncontacts; ++k) {
    if (m->contact_link[k] < 0 || m->contact_link[k] >= m->n)
      return cfail(SIM_ERR_INVALID_ARG, std::string(who) + ": contact_link out of range");
    tp->clink[k] = m->contact_link[k];
  }
  tp->nq = nq;
  tp->nv = nv;
  tp->nu = nu;
  tp->np = kParLink * m->n + kParSphere * m->ncontacts;
  return SIM_OK;
}

}  // namespace

extern "C" {

int sim_contact_param_count(const sim_contact_model* m, int* nq, int* nv, int* nu, int* nparams) {
  aba::clear_error();
  CTopo tp;
  const int rc = make_topo("sim_contact_param_count", m, &tp);
  if (rc) return rc;
  if (nq) *nq = tp.nq;
  if (nv) *nv = tp.nv;
  if (nu) *nu = tp.nu;
  if (nparams) *nparams = tp.np;
  return SIM_OK;
}

int sim_contact_flops(const sim_contact_model* m, const double* params, const double* q, const double* qd,
                      const double* tau, double dt, double* step_flops, double* grad_flops) {
  aba::clear_error();
  CTopo tp;
  const int rc = make_topo("sim_contact_flops", m, &tp);
  if (rc) return rc;
  if (!params || !q || !qd || (tp.nu > 0 && !tau) || !step_flops || !grad_flops)
    return cfail(SIM_ERR_INVALID_ARG, "sim_contact_flops: null argument");
  const Par<double> P{params, 1, 0};
  const int nx = tp.nq + tp.nv;
  {
    auto* w = new Work<CD>;
    CD x[kNX], x1[kNX], u[kNL];
    for (int k = 0; k < tp.nq; ++k) x[k] = CD(q[k]);
    for (int k = 0; k < tp.nv; ++k) x[tp.nq + k] = CD(qd[k]);
    for (int k = 0; k < tp.nu; ++k) u[k] = CD(tau[k]);
    g_cops = 0;
    contact_step(tp, P, x, x + tp.nq, u, dt, CD(tp.mu), x1, x1 + tp.nq, *w);
    *step_flops = (double)g_cops;
    delete w;
  }
  {
    // one reverse step: the recompute and the reverse statements
    auto* w = new Work<CD>;
    auto* rc = new Rec<CD>;
    auto* ad = new Adj<CD>;
    auto* art = new Art<CD>;
    CD x[kNX], xb[kNX], u[kNL], ub[kNL], mub(0.0);
    for (int k = 0; k < tp.nq; ++k) x[k] = CD(q[k]);
    for (int k = 0; k < tp.nv; ++k) x[tp.nq + k] = CD(qd[k]);
    for (int k = 0; k < tp.nu; ++k) u[k] = CD(tau[k]);
    for (int k = 0; k < nx; ++k) xb[k] = CD(1.0);
    g_cops = 0;
    contact_step_vjp(tp, P, x, x + tp.nq, u, dt, CD(tp.mu), xb, ub, mub, *w, *rc, *ad, *art);
    *grad_flops = (double)g_cops;
    delete w;
    delete rc;
    delete ad;
    delete art;
  }
  return SIM_OK;
}

int sim_contact_rollout(const sim_contact_model* m, int dtype, int batch, const void* params, const void* q0,
                        const void* qd0, const void* tau, double dt, int T, void* traj, void* qT, void* qdT,
                        int* ncontacts, void* stream) {
  aba::clear_error();
  CTopo tp;
  int rc = make_topo("sim_contact_rollout", m, &tp);
  if (rc) return rc;
  if (dtype != SIM_F32 && dtype != SIM_F64)
    return cfail(SIM_ERR_UNSUPPORTED_DTYPE, "sim_contact_rollout: dtype must be SIM_F32 or SIM_F64");
  if (batch < 0 || T < 0 || !(dt > 0))
    return cfail(SIM_ERR_INVALID_ARG, "sim_contact_rollout: need batch >= 0, T >= 0, dt > 0");
  if (batch == 0) return SIM_OK;
  if (!params || !q0 || !qd0 || !qT || !qdT || (T > 0 && tp.nu > 0 && !tau))
    return cfail(SIM_ERR_INVALID_ARG, "sim_contact_rollout: null array argument");
  hipError_t e;
  if (dtype == SIM_F64) {
    RollArgs<double> a{make_wave_topo(tp, false), batch, T, dt, (const double*)params, (const double*)q0, (const double*)qd0,
                       (const double*)tau, (double*)traj, (double*)qT, (double*)qdT, ncontacts};
    e = launch_rollout(a, (hipStream_t)stream);
  } else {
    RollArgs<float> a{make_wave_topo(constants_as_seen_by<float>(tp), false), batch, T, double((float)dt), (const float*)params, (const float*)q0, (const float*)qd0,
                      (const float*)tau, (float*)traj, (float*)qT, (float*)qdT, ncontacts};
    e = launch_rollout(a, (hipStream_t)stream);
  }
  if (e != hipSuccess) return cfail(SIM_ERR_HIP, std::string("sim_contact_rollout: launch failed: ") + hipGetErrorString(e));
  return SIM_OK;
}

int sim_contact_rollout_grad(const sim_contact_model* m, int dtype, int batch, const void* params, const void* traj,
                             const void* tau, double dt, int T, const void* gqT, const void* gqdT, void* gq0,
                             void* gqd0, void* gtau, void* gmu, void* stream) {
  aba::clear_error();
  CTopo tp;
  int rc = make_topo("sim_contact_rollout_grad", m, &tp);
  if (rc) return rc;
  if (dtype != SIM_F32 && dtype != SIM_F64)
    return cfail(SIM_ERR_UNSUPPORTED_DTYPE, "sim_contact_rollout_grad: dtype must be SIM_F32 or SIM_F64");
  if (batch < 0 || T < 0 || !(dt > 0))
    return cfail(SIM_ERR_INVALID_ARG, "sim_contact_rollout_grad: need batch >= 0, T >= 0, dt > 0");
  if (m->niter > kSweepMax)
    return cfail(SIM_ERR_INVALID_ARG, "sim_contact_rollout_grad: at most " + std::to_string(kSweepMax) +
                                          " PGS sweeps (niter) are recorded for the adjoint");
  if (batch == 0) return SIM_OK;
  if (!params || !traj || !gqT || !gqdT || !gq0 || !gqd0 || (T > 0 && tp.nu > 0 && (!tau || !gtau)))
    return cfail(SIM_ERR_INVALID_ARG, "sim_contact_rollout_grad: null array argument");
  hipError_t e;
  if (dtype == SIM_F64) {
    GradArgs<double> a{make_wave_topo(tp, true), batch, T, dt, (const double*)params, (const double*)traj, (const double*)tau,
                       (const double*)gqT, (const double*)gqdT, (double*)gq0, (double*)gqd0, (double*)gtau,
                       (double*)gmu};
    e = launch_grad(a, (hipStream_t)stream);
  } else {
    GradArgs<float> a{make_wave_topo(constants_as_seen_by<float>(tp), true), batch, T, double((float)dt), (const float*)params, (const float*)traj, (const float*)tau,
                      (const float*)gqT, (const float*)gqdT, (float*)gq0, (float*)gqd0, (float*)gtau,
                      (float*)gmu};
    e = launch_grad(a, (hipStream_t)stream);
  }
  if (e != hipSuccess)
    return cfail(SIM_ERR_HIP, std::string("sim_contact_rollout_grad: launch failed: ") + hipGetErrorString(e));
  return SIM_OK;
}

int sim_contact_autotune(const sim_contact_model* m, int dtype, int batch, const void* params, const void* q0,
                         const void* qd0, const void* tau, double dt, int T_probe, void* stream,
                         sim_contact_tiling_t* chosen, double* rollout_ms, double* grad_ms) {
  aba::clear_error();
  CTopo tp;
  int rc = make_topo("sim_contact_autotune", m, &tp);
  if (rc) return rc;
  if (dtype != SIM_F32 && dtype != SIM_F64)
    return cfail(SIM_ERR_UNSUPPORTED_DTYPE, "sim_contact_autotune: dtype must be SIM_F32 or SIM_F64");
  if (batch < 1 || T_probe < 1 || !(dt > 0))
    return cfail(SIM_ERR_INVALID_ARG, "sim_contact_autotune: need batch >= 1, T_probe >= 1, dt > 0");
  if (m->niter > kSweepMax)
    return cfail(SIM_ERR_INVALID_ARG, "sim_contact_autotune: at most " + std::to_string(kSweepMax) +
                                          " PGS sweeps (niter) are recorded for the adjoint");
  if (!params || !q0 || !qd0 || (tp.nu > 0 && !tau) || !chosen)
    return cfail(SIM_ERR_INVALID_ARG, "sim_contact_autotune: null argument");
  const hipStream_t st = (hipStream_t)stream;
  const size_t es = dtype == SIM_F64 ? sizeof(double) : sizeof(float);
  const size_t B = (size_t)batch, T = (size_t)T_probe, nq = tp.nq, nv = tp.nv, nu = tp.nu;
  // probe buffers: traj, qT, qdT, gq0, gqd0, gtau, and the zero seeds gqT, gqdT
  const size_t n_traj = (T + 1) * (nq + nv) * B, n_tau = T * nu * B;
  const size_t total = (n_traj + 2 * (nq + nv) * B + n_tau + (nq + nv) * B) * es;
  char* buf = nullptr;
  if (hipMalloc(&buf, total) != hipSuccess) return cfail(SIM_ERR_HIP, "sim_contact_autotune: probe allocation failed");
  char* p = buf;
  auto take = [&](size_t n) { char* r = p; p += n * es; return r; };
  void* traj = take(n_traj);
  void* qT = take(nq * B);
  void* qdT = take(nv * B);
  void* gq0 = take(nq * B);
  void* gqd0 = take(nv * B);
  void* gtau = take(n_tau);
  void* gqT = take(nq * B);
  void* gqdT = take(nv * B);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  sim_contact_model mm = *m;
  mm.tiling = nullptr;
  float ms_r = 0.f, ms_g = 0.f;
  rc = SIM_OK;
  do {
    if (hipMemsetAsync(gqT, 0, (nq + nv) * B * es, st) != hipSuccess || hipEventCreate(&e0) != hipSuccess ||
        hipEventCreate(&e1) != hipSuccess) {
      rc = cfail(SIM_ERR_HIP, "sim_contact_autotune: set-up failed");
      break;
    }
    // once untimed, then once between events
    auto timed = [&](auto&& run, float* ms) -> int {
      int r = run();
      if (r) return r;
      if (hipEventRecord(e0, st) != hipSuccess) return cfail(SIM_ERR_HIP, "sim_contact_autotune: event failed");
      r = run();
      if (r) return r;
      if (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
          hipEventElapsedTime(ms, e0, e1) != hipSuccess)
        return cfail(SIM_ERR_HIP, "sim_contact_autotune: timing failed");
      return SIM_OK;
    };
    rc = timed([&] { return sim_contact_rollout(&mm, dtype, batch, params, q0, qd0, tau, dt, T_probe, traj, qT, qdT,
                                                nullptr, stream); }, &ms_r);
    if (!rc)
      rc = timed([&] { return sim_contact_rollout_grad(&mm, dtype, batch, params, traj, tau, dt, T_probe, gqT, gqdT,
                                                       gq0, gqd0, gtau, nullptr, stream); }, &ms_g);
  } while (false);
  (void)hipStreamSynchronize(st);
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipFree(buf);
  if (rc) return rc;
  *chosen = {kRollSplDefault, kGradSplDefault, 1};
  if (rollout_ms) *rollout_ms = ms_r / T_probe;
  if (grad_ms) *grad_ms = ms_g / T_probe;
  return SIM_OK;
}

}  // extern "C"
