// The method's device-resident state and scalar steps, shared by every kernel
// of the library: the pairwise wave reduction (DPP), and the scalar step that
// ends each reduction phase (stopping test, alpha, beta, omega).  Every thread
// evaluates a scalar step on identical inputs; only the leader writes the
// history.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pbcgs {

constexpr int kWG = 256;                  // threads per workgroup: 4 x wave64
constexpr int kMaxD = 5;                  // dot products per reduction phase
constexpr int kMaxR = 1024;               // 64-row blocks per wave (a power of two)
constexpr int kLevels = 11;               // levels of a wave's pairwise tree: kMaxR = 2^(kLevels-1)
constexpr int kMaxG = 1024;               // workgroups of a producing kernel
constexpr int kChunk = kMaxG / kWG;       // partials per thread when consuming

// DS_CHECK (precision form only): the binary32 recursive residual passed tol;
// the host confirms with the binary64 true residual before declaring SUCCESS.
enum : int32_t { DS_RUNNING = 0, DS_SUCCESS = 1, DS_BREAKDOWN = 2, DS_NONFINITE = 3, DS_CHECK = 4 };

// Device-resident solver state: scalars of the method and the status word.
struct alignas(128) DevState {
  double alpha;   // alpha_i
  double beta;    // beta_{i-1}
  double omega;   // omega_{i-1} (omega_i once reduction 1 of iteration i is done)
  double gamma;   // (r0, r_i)
  double rho0;    // ||r_0||
  double relres;  // last ||r_i|| / ||r_0||
  double tol;
  double result;  // output of utility reductions
  int32_t status;
  int32_t iters;  // completed x updates
  int32_t n_rr;   // residual replacements done
  int32_t pad[5];
};

// ---------------------------------------------------------------------------
// Pairwise reduction machinery.
// ---------------------------------------------------------------------------

// 64-bit DPP move: lane l receives the value of the lane CTRL selects, or 0
// where there is none.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

template <int CTRL, class T>
__device__ __forceinline__ T dpp_t(T v) {
  if constexpr (sizeof(T) == 8) return dpp_f64<CTRL>(v);
  else return dpp_f32<CTRL>(v);
}

// Balanced-tree sum over the 64 lanes of a wave; the result is valid in lane
// 63.  Level m adds to the last lane of every aligned block of 2m lanes the
// sum held by the last lane of the block's left half (row_shr 1, 2, 4, 8,
// then row_bcast 15 and 31 across the 16-lane rows), so lane 63 ends with
// ((l0 + l1) + (l2 + l3)) + ... exactly as the pairwise order prescribes.  The
// other lanes' values do not reach lane 63 and are not masked off: a masked
// DPP move needs its destination zeroed first, which made every 64-bit step
// five instructions instead of three.
template <int ND, class T>
__device__ __forceinline__ void wave_sum63(T (&v)[ND]) {
#pragma unroll
  for (int k = 0; k < ND; ++k) v[k] = v[k] + dpp_t<0x111>(v[k]);
#pragma unroll
  for (int k = 0; k < ND; ++k) v[k] = v[k] + dpp_t<0x112>(v[k]);
#pragma unroll
  for (int k = 0; k < ND; ++k) v[k] = v[k] + dpp_t<0x114>(v[k]);
#pragma unroll
  for (int k = 0; k < ND; ++k) v[k] = v[k] + dpp_t<0x118>(v[k]);
#pragma unroll
  for (int k = 0; k < ND; ++k) v[k] = v[k] + dpp_t<0x142>(v[k]);
#pragma unroll
  for (int k = 0; k < ND; ++k) v[k] = v[k] + dpp_t<0x143>(v[k]);
}

__device__ __forceinline__ bool finite(double v) { return __builtin_isfinite(v); }
__device__ __forceinline__ bool leader() { return blockIdx.x == 0 && threadIdx.x == 0; }

// Register copy of the state (field by field: no aligned aggregate on the stack).
struct State {
  double alpha, beta, omega, gamma, rho0, relres, tol, result;
  int32_t status, iters, n_rr;
};

__device__ __forceinline__ State load_state(const DevState* p) {
  State s;
  s.alpha = p->alpha; s.beta = p->beta; s.omega = p->omega; s.gamma = p->gamma;
  s.rho0 = p->rho0; s.relres = p->relres; s.tol = p->tol; s.result = p->result;
  s.status = p->status; s.iters = p->iters; s.n_rr = p->n_rr;
  return s;
}

__device__ __forceinline__ void store_state(DevState* p, const State& s) {
  p->alpha = s.alpha; p->beta = s.beta; p->omega = s.omega; p->gamma = s.gamma;
  p->rho0 = s.rho0; p->relres = s.relres; p->tol = s.tol; p->result = s.result;
  p->status = s.status; p->iters = s.iters; p->n_rr = s.n_rr;
}

// ---------------------------------------------------------------------------
// Scalar steps of the method.  Every thread evaluates them on identical
// inputs; only the leader writes the history.
// ---------------------------------------------------------------------------

// gamma = (r0, r0), rho0 = ||r0|| (the setup of Algorithms 7-11).
__device__ __forceinline__ void fin_setup_gamma(State& s, double* hist, double g) {
  s.gamma = g;
  const double rho0 = sqrt(g);
  s.rho0 = rho0;
  s.relres = 1.0;
  if (hist && leader()) hist[0] = 1.0;
  if (!finite(rho0)) s.status = DS_NONFINITE;
  else if (rho0 == 0.0) { s.status = DS_SUCCESS; s.relres = 0.0; }
}

// alpha_0 = (r0, r0) / (r0, w0), beta_{-1} = omega_{-1} = 0 (the setup of Algorithms 9 and 11).
__device__ __forceinline__ void fin_setup_alpha(State& s, double delta) {
  if (!finite(delta)) { s.status = DS_NONFINITE; return; }
  if (delta == 0.0) { s.status = DS_BREAKDOWN; return; }
  const double alpha = s.gamma / delta;
  if (!finite(alpha)) { s.status = DS_NONFINITE; return; }
  s.alpha = alpha;
  s.beta = 0.0;
  s.omega = 0.0;
}

// omega_i = (q, y) / (y, y)  (reduction 1 of Algorithms 7, 9, 10 and 11).
// Returns true when (y, y) = 0: then q = 0
// and x_i + alpha_i p^_i is the solution; the caller applies that update.
__device__ __forceinline__ bool fin_omega(State& s, double* hist, double qy, double yy) {
  if (!finite(qy) || !finite(yy)) { s.status = DS_NONFINITE; return false; }
  if (yy == 0.0) {
    s.iters += 1;
    s.relres = 0.0;
    if (hist && leader()) hist[s.iters] = 0.0;
    s.status = DS_SUCCESS;
    return true;
  }
  const double omega = qy / yy;
  if (!finite(omega)) { s.status = DS_NONFINITE; return false; }
  s.omega = omega;
  return false;
}

// alpha_{i+1} of the pipelined solvers from gamma' = (r0, r_{i+1}), eta = (r0, w_{i+1}),
// sigma_s = (r0, s_i), sigma_z = (r0, z_i): eq. (3) is gamma' / (eta + beta sigma_s
// - beta omega sigma_z); eq. (5) is the same quantity rearranged so that sigma_s
// drops out, (1/omega + eta/gamma' - (beta omega) (sigma_z/gamma'))^{-1}.  Both
// evaluate in the order and grouping the equations write, without contraction.
__device__ __forceinline__ void next_alpha(State& s, int32_t aform, double g1, double eta, double sig_s,
                                           double sig_z, double beta, double omega) {
  double an;
  if (aform == 5) {
    if (g1 == 0.0) { s.status = DS_BREAKDOWN; return; }
    const double den = (1.0 / omega + eta / g1) - (beta * omega) * (sig_z / g1);
    if (den == 0.0) { s.status = DS_BREAKDOWN; return; }
    an = 1.0 / den;
  } else {
    const double den = eta + beta * sig_s - beta * omega * sig_z;
    if (den == 0.0 || g1 == 0.0) { s.status = DS_BREAKDOWN; return; }
    an = g1 / den;
  }
  if (!finite(an)) { s.status = DS_NONFINITE; return; }
  s.alpha = an;
  s.gamma = g1;
}

// Reduction 2 of p-BiCGStab: stopping test, beta_i and alpha_{i+1} by eq. (3)
// or eq. (5) (Algorithm 9, Algorithm 11).
__device__ __forceinline__ void fin_pipe_b(State& s, double* hist, const double (&d)[5], int32_t aform) {
  const double g1 = d[0], eta = d[1], sig_s = d[2], sig_z = d[3], nu = d[4];
  s.iters += 1;
  if (!finite(g1) || !finite(eta) || !finite(sig_s) || !finite(sig_z) || !finite(nu)) {
    s.status = DS_NONFINITE;
    return;
  }
  const double relres = sqrt(nu) / s.rho0;
  s.relres = relres;
  if (hist && leader()) hist[s.iters] = relres;
  if (relres <= s.tol) { s.status = DS_SUCCESS; return; }
  const double alpha = s.alpha, omega = s.omega, gamma = s.gamma;
  if (omega == 0.0 || gamma == 0.0) { s.status = DS_BREAKDOWN; return; }
  const double beta = (alpha / omega) * (g1 / gamma);
  if (!finite(beta)) { s.status = DS_NONFINITE; return; }
  s.beta = beta;
  next_alpha(s, aform, g1, eta, sig_s, sig_z, beta, omega);
}

// alpha_i = (r0, r_i) / (r0, s_i)  (the first reduction of Algorithm 7).
__device__ __forceinline__ void fin_bicg_alpha(State& s, double delta) {
  if (!finite(delta)) { s.status = DS_NONFINITE; return; }
  if (delta == 0.0) { s.status = DS_BREAKDOWN; return; }
  const double alpha = s.gamma / delta;
  if (!finite(alpha)) { s.status = DS_NONFINITE; return; }
  s.alpha = alpha;
}

// Stopping test and beta_i = (alpha/omega) (r0, r_{i+1}) / (r0, r_i)  (the last reduction of Algorithm 7).
__device__ __forceinline__ void fin_bicg_beta(State& s, double* hist, double g1, double nu) {
  s.iters += 1;
  if (!finite(g1) || !finite(nu)) { s.status = DS_NONFINITE; return; }
  const double relres = sqrt(nu) / s.rho0;
  s.relres = relres;
  if (hist && leader()) hist[s.iters] = relres;
  if (relres <= s.tol) { s.status = DS_SUCCESS; return; }
  const double alpha = s.alpha, omega = s.omega, gamma = s.gamma;
  if (omega == 0.0 || gamma == 0.0) { s.status = DS_BREAKDOWN; return; }
  const double beta = (alpha / omega) * (g1 / gamma);
  if (!finite(beta)) { s.status = DS_NONFINITE; return; }
  s.beta = beta;
  s.gamma = g1;
}

// First reduction of Algorithms 4 and 6: rho0 = sqrt(nu_0), alpha_0 = gamma_0 / delta_0, beta_0 = 0.
__device__ __forceinline__ void fin_cgs_first(State& s, double* hist, const double (&d)[3]) {
  const double gamma = d[0], delta = d[1], nu = d[2];
  s.relres = 1.0;
  if (hist && leader()) hist[0] = 1.0;
  if (!finite(gamma) || !finite(delta) || !finite(nu)) { s.status = DS_NONFINITE; return; }
  const double rho0 = sqrt(nu);
  s.rho0 = rho0;
  if (rho0 == 0.0) { s.status = DS_SUCCESS; s.relres = 0.0; return; }
  if (delta == 0.0) { s.status = DS_BREAKDOWN; return; }
  const double alpha = gamma / delta;
  if (!finite(alpha)) { s.status = DS_NONFINITE; return; }
  s.alpha = alpha;
  s.beta = 0.0;
  s.gamma = gamma;
}

// Later reductions of Algorithms 4 and 6: stopping test on ||r_i|| (i = s.iters),
// beta_i = gamma_i / gamma_{i-1}, alpha_i = (delta / gamma_i - beta_i / alpha_{i-1})^{-1}.
__device__ __forceinline__ void fin_cgs_next(State& s, double* hist, const double (&d)[3]) {
  const double g1 = d[0], delta = d[1], nu = d[2];
  if (!finite(g1) || !finite(delta) || !finite(nu)) { s.status = DS_NONFINITE; return; }
  const double relres = sqrt(nu) / s.rho0;
  s.relres = relres;
  if (hist && leader()) hist[s.iters] = relres;
  if (relres <= s.tol) { s.status = DS_SUCCESS; return; }
  if (s.gamma == 0.0 || g1 == 0.0 || s.alpha == 0.0) { s.status = DS_BREAKDOWN; return; }
  const double beta = g1 / s.gamma;
  if (!finite(beta)) { s.status = DS_NONFINITE; return; }
  const double den = delta / g1 - beta / s.alpha;
  if (den == 0.0) { s.status = DS_BREAKDOWN; return; }
  const double alpha = 1.0 / den;
  if (!finite(alpha)) { s.status = DS_NONFINITE; return; }
  s.beta = beta;
  s.alpha = alpha;
  s.gamma = g1;
}

// alpha = gamma / (s, p) (Algorithm 2).
__device__ __forceinline__ void fin_cg_alpha(State& s, double delta) {
  if (!finite(delta)) s.status = DS_NONFINITE;
  else if (delta == 0.0) s.status = DS_BREAKDOWN;
  else {
    const double alpha = s.gamma / delta;
    if (!finite(alpha)) s.status = DS_NONFINITE;
    else s.alpha = alpha;
  }
}

// Algorithm 2, kernel 3: stopping test, beta = (r', u') / (r, u) ; p = u + beta p.
__device__ __forceinline__ void fin_cg_beta(State& s, double* hist, const double (&d)[2]) {
  const double g1 = d[0], nu = d[1];
  s.iters += 1;
  if (!finite(g1) || !finite(nu)) { s.status = DS_NONFINITE; return; }
  const double relres = sqrt(nu) / s.rho0;
  s.relres = relres;
  if (hist && leader()) hist[s.iters] = relres;
  if (relres <= s.tol) { s.status = DS_SUCCESS; return; }
  if (s.gamma == 0.0) { s.status = DS_BREAKDOWN; return; }
  const double beta = g1 / s.gamma;
  if (!finite(beta)) { s.status = DS_NONFINITE; return; }
  s.beta = beta;
  s.gamma = g1;
}

}  // namespace pbcgs
