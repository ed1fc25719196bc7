// Internal declarations of the HIP library: argument blocks, device helpers
// and kernel launchers.  Not part of the public ABI (include/lasp.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lasp {

constexpr double kCkms = 299792.458;            // speed of light, km/s
constexpr double kLn10 = 2.302585092994045684;  // ln 10
constexpr float kSigmaFloorPx = 0.1f;           // lower bound of the kernel width, pixels
constexpr int kNB = 20;                         // interpolator terms (cubic in 3 coordinates)
constexpr int kMaxClasses = 3;                  // emulator temperature classes
constexpr int kNP = 5;                          // free parameters per spectrum
constexpr int kNPL = 17;                        // pixels owned by one lane in the fused pass
constexpr int kTB = 8;                          // taps per register block
constexpr int kMaxArms = 4;

// Status bits (same values as LASP_ST_* in lasp.h).
constexpr uint32_t kStNonfinite = 0x01u;
constexpr uint32_t kStNoData = 0x02u;
constexpr uint32_t kStSingular = 0x04u;
constexpr uint32_t kStContNonpos = 0x08u;
constexpr uint32_t kStOutOfBox = 0x10u;
constexpr uint32_t kStSigmaFloor = 0x20u;
constexpr uint32_t kStStopFlat = 0x40u;
constexpr uint32_t kStStopRising = 0x80u;
constexpr uint32_t kStNotConverged = 0x100u;
constexpr uint32_t kStPolishLimit = 0x200u;
constexpr int kMaxStopWindow = 4096;

// Levenberg-Marquardt polish: a spectrum stops when the predicted chi2
// decrease of its next step is below kLmDecreaseTol (chi2 units: the
// remaining improvement is 1e-3 standard deviations in any direction), when
// an accepted step lowers chi2 by less than kLmDropTol relative or moves u
// by less than kLmStepTol, or when the damping passes kLmLambdaMax.
constexpr double kLmDecreaseTol = 1e-6;
constexpr double kLmDropTol = 1e-10;
constexpr double kLmStepTol = 1e-7;
constexpr double kLmLambdaMax = 1e10;

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// Geometry shared by every per-step kernel.
struct Geometry {
  int B;        // spectra
  int P;        // pixels
  int M;        // margin
  int Pe;       // P + 2M basis columns
  int ldF;      // row stride of F' / F-bar' / padded basis (>= Pe; a multiple of 128: the adjoint
                // contractions and the fit's Phi-bar split it into eight parts of 16-column blocks)
  int nd;       // continuum coefficients D + 1
  int block;    // threads of the fused pass
  int n_arms;   // >= 1
  int arm_start[kMaxArms + 1];  // arm a covers pixels [arm_start[a], arm_start[a+1])
  double arm_sig2[kMaxArms];    // instrumental sigma^2, (km/s)^2 (0 for a single bare arm)
  int bare;                     // 1: one arm without instrument term
  double inv_scale;             // pixels per km/s = 1 / (c ln10 dlog10)
  double rv_lo, rv_half;        // RV = rv_lo + (u4 + 1) rv_half
  double sg_lo, sg_half;        // sigma = sg_lo + (u5 + 1) sg_half
  int n_classes;                // 1, or 3 emulator temperature classes
  int nb;                       // basis rows: kNB * n_classes
  double lt_lo, lt_half;        // log10 Teff = lt_lo + (u1 + 1) lt_half
  double edges[4];              // Teff regime edges (K) of the class blend
  double hpow[11];              // h^n, h = 2 / P: pixel step of the continuum's x
};

// Per-spectrum state and scratch owned by the library.
struct State {
  float *u;         // [B][5] normalised parameters
  float *m;         // [B][5] Adam first moment
  float *v;         // [B][5] Adam second moment
  int *t;           // [B] Adam step count
  int *target;      // [B] step count at which a slot stops (NULL: every slot runs)
  float2 *ow;       // [B][kNPL][block] (o/w, W w^2) in lane-major order
  float *wscale;    // [B] flux weight w
  int *neff;        // [B]
  uint32_t *status; // [B]
  float *fp;        // [B][ldF] (or [B][4][ldF]) F'
  int fp_stride;    // floats between consecutive spectra in fp (ldF or 4 ldF)
  float *fbar;      // [B][ldF] F-bar'
  float *g45;       // [B][2] dJ/du4, dJ/du5
  double *chi2;     // [B]
  double *lhist;    // [B][stop window] loss history ring (stopping rules)
  int *nrise;       // [B] consecutive steps at which the loss rose
  // Optional list of the spectra still taking steps (stopping rules on):
  // the per-step kernels then work on order[0 .. *n_active) instead of
  // 0 .. B.  NULL: every spectrum, in index order.
  const int *order;     // [B] spectrum indices, active ones first
  const int *n_active;  // [1] length of the list
  float *basis;     // [nb][ldF] zero-padded copy of the basis
  uint16_t *basis_hi;  // 20 x ldF, bf16 high part in operand order (BF16x3, adjoint contraction)
  uint16_t *basis_lo;  // 20 x ldF, bf16 low part
  uint16_t *basis_thi; // 32 x ldF, bf16 high part in operand order, rows 1..19 (forward)
  uint16_t *basis_tlo; // 32 x ldF, bf16 low part
};

// Inputs and outputs of the Clean mask kernel.  obs, ivar and model are
// [B][P] row-major in the units of obs.  With s.ow set, the kernel writes
// the new weights into the fused pass's (o/w, W w^2) array and n_eff; with
// s.target set, stopped spectra are skipped.
struct CleanArgs {
  const float *obs;
  const float *ivar;
  const float *model;
  float f_shift;
  uint8_t *keep_out;   // optional [B][P]: 1 kept, 0 clipped
  int32_t *masked_out; // optional [B]: clipped valid pixels
  State s;             // ow, wscale, neff, t, target (others unused)
};

// Inputs and outputs of a one-shot evaluation's fused pass, which prepares
// its spectra itself.
struct OneShot {
  const float *obs;   // [B][P]
  const float *ivar;  // [B][P]
  float quantile;     // of the flux weight
  int write_ow;       // 1: leave (o/w, W w^2) in s.ow for a later kernel
  float *J;           // optional [B]
};

// Arguments of the covariance kernel.
struct CovArgs {
  double lo[kNP], hi[kNP];  // normalisation box
  OneShot os;               // one-shot evaluation: inputs and J (write_ow unused)
  int set_status;           // 1: write chi2 and the evaluation's status
  float *model_out;         // optional [B][P]
  float *out_jac;           // optional [B][5][P]
  double *out_cov;          // optional [B][5][5]
  int last;                 // polish: iterations at most
};

struct AdamCfg {
  float lr, beta1, beta2, eps;
  int stop_window;  // 0: fixed step count
  float stop_tol;
};

// ---------------------------------------------------------------- host side
hipError_t launch_prepare(const Geometry &g, const State &s, const float *obs, const float *ivar,
                          const float *init_params, const double *box_lo, const double *box_hi,
                          float weight_quantile, int init_state, int target_steps, hipStream_t st);

// A spectrum takes Adam steps while t < target (always when target is NULL).
#ifdef __HIPCC__
__device__ inline bool slot_active(const State &s, int spec) {
  return s.target == nullptr || s.t[spec] < s.target[spec];
}
// Entries the per-step kernels cover, and the spectrum of entry i.
__device__ inline int work_count(const Geometry &g, const State &s) {
  return s.order ? *s.n_active : g.B;
}
__device__ inline int work_spec(const State &s, int i) { return s.order ? s.order[i] : i; }
#endif
// Writes the spectra with slot_active true to order -- in index order, or
// with several emulator classes in index order within each Teff regime,
// regimes by increasing Teff -- and their number to n_active (one
// workgroup).
hipError_t launch_compact(const Geometry &g, const State &s, int *order, int *n_active,
                          hipStream_t st);
hipError_t launch_interp_fwd(const Geometry &g, const State &s, int deriv_rows, int bf16x3,
                             hipStream_t st);
// set_status: 1 for a pass at the parameters a call returns (the
// evaluation bits of the status are replaced), 0 for the passes of the
// steps (status untouched).
// An adjoint pass is that of an Adam step: model_out NULL, set_status 0.
hipError_t launch_fused(const Geometry &g, const State &s, int adjoint, float *model_out,
                        int set_status, hipStream_t st);
// The same pass with the preparation of each spectrum in it, for an
// evaluation at fixed parameters: writes chi2, n_eff, the flux weight and the
// whole status.
hipError_t launch_fused_oneshot(const Geometry &g, const State &s, int adjoint, float *model_out,
                                const OneShot &os, hipStream_t st);
// n_steps further Adam steps of every spectrum, one workgroup each (one emulator
// class, FP32 contractions, no stopping rules): the results of as many
// launches of the three step kernels, bit for bit.
hipError_t launch_fit(const Geometry &g, const State &s, const AdamCfg &adam, int n_steps,
                      hipStream_t st);
hipError_t launch_interp_bwd(const Geometry &g, const State &s, const AdamCfg *adam,
                             float *grad_out, int bf16x3, hipStream_t st);
hipError_t launch_split_basis(const Geometry &g, const State &s, hipStream_t st);
hipError_t launch_finalize(const Geometry &g, const State &s, const double *box_lo,
                           const double *box_hi, float *out_params, uint32_t *status_out,
                           double *chi2_out, int32_t *steps_out, hipStream_t st);
// Outputs of a forward evaluation out of the scratch (each may be NULL).
hipError_t launch_outputs(const Geometry &g, const State &s, double *chi2_out, float *J_out,
                          int32_t *neff_out, uint32_t *status_out, hipStream_t st);
hipError_t launch_progress(const Geometry &g, const State &s, int32_t *steps, int32_t *done,
                           hipStream_t st);
// Evaluation with covariance and/or model Jacobian (s.fp: four rows per
// spectrum): of prepared spectra, or preparing them from ca.os.
hipError_t launch_cov(const Geometry &g, const State &s, const CovArgs &ca, hipStream_t st);
hipError_t launch_cov_oneshot(const Geometry &g, const State &s, const CovArgs &ca,
                              hipStream_t st);
// Levenberg-Marquardt polish of prepared spectra from s.u (s.fp: scratch of
// four rows per spectrum), each until its own stop or ca.last iterations.
hipError_t launch_lm(const Geometry &g, const State &s, const CovArgs &ca, hipStream_t st);
hipError_t launch_clean(const Geometry &g, const CleanArgs &a, hipStream_t st);
hipError_t launch_resample(const float *src, int n_rows, int n_src, int64_t ld_src, double lam0,
                           double dlam, float *out, int n_out, int64_t ld_out, double lg0,
                           double dlog10, hipStream_t st);
bool fused_supported(int block, int nd);
// Sets the calling thread's lasp_last_error() message; returns code.
int set_error(int code, const char *msg);
size_t fused_smem_bytes(const Geometry &g);

// [x^n] T_k(x) for k, n <= 10, from T_k = 2x T_{k-1} - T_{k-2}.
struct ChebPow {
  int c[11][11];
};
constexpr ChebPow make_cheb_pow() {
  ChebPow t{};
  t.c[0][0] = 1;
  t.c[1][1] = 1;
  for (int k = 2; k < 11; ++k)
    for (int n = 0; n <= k; ++n) t.c[k][n] = (n > 0 ? 2 * t.c[k - 1][n - 1] : 0) - t.c[k - 2][n];
  return t;
}
constexpr ChebPow kChebPow = make_cheb_pow();

// ---- Nodes of the continuum moments ---------------------------------------
constexpr int kMid = kNPL / 2;  // a lane's middle pixel: local expansions are about j0 + kMid

// A lane's 17 pixels span so little of the row that every polynomial the
// moments need is, on them, its own interpolant at a few nodes.  For nodes
// x_mid + h tau_c (tau_c the seven Chebyshev points of [-8, 8] pixels, h = 2 / P)
//   sum_i y_i p(x_i) = sum_c Y_c p(x_mid + h tau_c),  Y_c = sum_i L_c(t_i) y_i
// up to the interpolation error of p.  The nodes are three pairs +-tau_c and
// the middle, so the Lagrange weights fold into sums and differences of the
// pixels at +-t:
//   Y_+-c = sum_t E_c(t) (y_t + y_-t) +- sum_t O_c(t) (y_t - y_-t).
constexpr int kNodes = 7, kPairs = kNodes / 2;
struct MomentNodes {
  double tau[kPairs] = {};
  float e[kPairs + 1][kMid + 1] = {}, o[kPairs][kMid + 1] = {};  // e[kPairs]: the middle
};
constexpr MomentNodes make_moment_nodes() {
  // cos((2 c - 1) pi / 14), c = 1, 2, 3
  constexpr double cosines[kPairs] = {0.974927912181823607, 0.781831482468029809,
                                      0.433883739117558120};
  MomentNodes n{};
  for (int c = 0; c < kPairs; ++c) n.tau[c] = kMid * cosines[c];
  for (int c = 0; c <= kPairs; ++c)
    for (int t = 0; t <= kMid; ++t) {
      const bool mid = c == kPairs;
      const double tc = mid ? 0.0 : n.tau[c];
      double v = 1.0;  // the factors of the other pairs
      for (int d = 0; d < kPairs; ++d)
        if (d != c) v *= (t * t - n.tau[d] * n.tau[d]) / (tc * tc - n.tau[d] * n.tau[d]);
      n.e[c][t] = (float)(mid ? v : 0.5 * v * t * t / (tc * tc));
      if (!mid) n.o[c][t] = (float)(0.5 * v * t / tc);
    }
  return n;
}
inline constexpr MomentNodes kMomentNodes = make_moment_nodes();

// Whether the nodes hold the moments' polynomials (degree n = 2 (nd - 1)) to
// 1e-7 of their largest value on any lane of a row of P pixels: the Chebyshev
// interpolation error 2 (a / 2)^7 |p^(7)| / 7!, a = 16 / P.  The last lane's
// nodes reach up to d = 30 / P past the row's end, and there a derivative of a
// polynomial of degree n bounded by one on the row is at most T_n's: the sum
// of T_n^(7 + m)(1) d^m / m! with T_n^(k)(1) = prod_{i < k} (n^2 - i^2) /
// (2 i + 1).  Degree 10: 1,965 pixels and more, 8: 1,229, 6: 656, 4: 242;
// shorter rows sum over the pixels.  (Six nodes would serve 3,818 pixels and
// more at degree 10; the step's pass measured 0.290 ms with six, 0.293
// with seven and 0.321 with both in one kernel, 16,384 x 3,900.)
inline bool moment_nodes_hold(int nd, int P) {
  const int n = 2 * (nd - 1);
  const double a = 16.0 / (double)P, d = 30.0 / (double)P;
  auto step = [&](int k) { return ((double)n * n - (double)k * k) / (2.0 * k + 1.0); };
  double term = 1.0, b = 0.0;
  for (int k = 0; k < kNodes; ++k) term *= step(k);
  for (int k = kNodes; k <= n; ++k) {  // term: T_n^(k)(1) d^m / m!, m = k - 7
    b += term;
    term *= step(k) * d / (double)(k - kNodes + 1);
  }
  b *= 2.0;
  for (int k = 0; k < kNodes; ++k) b *= 0.5 * a / (k + 1.0);
  return b <= 1e-7;
}

// -------------------------------------------------------------- device side
#ifdef __HIPCC__

// OUT_OF_BOX of the parameters u (|u_t| > 1.5 for some t, or not finite).
__device__ inline uint32_t box_bit(const float *u) {
  uint32_t b = 0;
  for (int t = 0; t < kNP; ++t)
    if (!(fabsf(u[t]) <= 1.5f)) b = kStOutOfBox;
  return b;
}

// Eq. 1 features: monomials of total degree <= 3 in x = (u1, u2, u3),
// graded lexicographic order.
__device__ inline void features(float x, float y, float z, float *phi) {
  phi[0] = 1.f;
  phi[1] = x; phi[2] = y; phi[3] = z;
  phi[4] = x * x; phi[5] = x * y; phi[6] = x * z; phi[7] = y * y; phi[8] = y * z; phi[9] = z * z;
  phi[10] = x * x * x; phi[11] = x * x * y; phi[12] = x * x * z; phi[13] = x * y * y;
  phi[14] = x * y * z; phi[15] = x * z * z; phi[16] = y * y * y; phi[17] = y * y * z;
  phi[18] = y * z * z; phi[19] = z * z * z;
}

// Weights of the three emulator classes (cool, warm, hot) at u1 (Eq. 1 over
// the five Teff regimes): with a = clamp((T - e0) / (e1 - e0)) and
// b = clamp((T - e2) / (e3 - e2)) the weights are 1 - a, a (1 - b) and a b,
// so one class holds inside a regime and two blend linearly in Teff across a
// transition regime.  dw = d w / d u1 (zero where the blend is flat).  FP64
// inside, FP32 out.
__device__ inline void class_weights(const Geometry &g, float u1, float *w, float *dw) {
  const double lt = g.lt_lo + ((double)u1 + 1.0) * g.lt_half;
  const double T = exp(kLn10 * lt);
  const double dT = T * kLn10 * g.lt_half;
  const double w01 = g.edges[1] - g.edges[0], w23 = g.edges[3] - g.edges[2];
  double a = (T - g.edges[0]) / w01, da = dT / w01;
  if (!(T > g.edges[0] && T < g.edges[1])) da = 0.0;
  a = fmin(fmax(a, 0.0), 1.0);
  double b = (T - g.edges[2]) / w23, db = dT / w23;
  if (!(T > g.edges[2] && T < g.edges[3])) db = 0.0;
  b = fmin(fmax(b, 0.0), 1.0);
  w[0] = (float)(1.0 - a);
  w[1] = (float)(a * (1.0 - b));
  w[2] = (float)(a * b);
  dw[0] = (float)(-da);
  dw[1] = (float)(da * (1.0 - b) - a * db);
  dw[2] = (float)(da * b + a * db);
}

// d phi_k / d x_t for t = 0, 1, 2 (d[t][k]).
__device__ inline void feature_derivs(float x, float y, float z, float (*d)[kNB]) {
#pragma unroll
  for (int t = 0; t < 3; ++t)
#pragma unroll
    for (int k = 0; k < kNB; ++k) d[t][k] = 0.f;
  d[0][1] = 1.f; d[1][2] = 1.f; d[2][3] = 1.f;
  d[0][4] = 2.f * x;
  d[0][5] = y; d[1][5] = x;
  d[0][6] = z; d[2][6] = x;
  d[1][7] = 2.f * y;
  d[1][8] = z; d[2][8] = y;
  d[2][9] = 2.f * z;
  d[0][10] = 3.f * x * x;
  d[0][11] = 2.f * x * y; d[1][11] = x * x;
  d[0][12] = 2.f * x * z; d[2][12] = x * x;
  d[0][13] = y * y; d[1][13] = 2.f * x * y;
  d[0][14] = y * z; d[1][14] = x * z; d[2][14] = x * y;
  d[0][15] = z * z; d[2][15] = 2.f * x * z;
  d[1][16] = 3.f * y * y;
  d[1][17] = 2.f * y * z; d[2][17] = y * y;
  d[1][18] = z * z; d[2][18] = 2.f * y * z;
  d[2][19] = 3.f * z * z;
}

// Feature row t of spectrum s: t = 0 is phi(u), t = 1..3 is d phi / d u_t.
__device__ inline void feature_row(const float *u, int t, float *out) {
  const float x = u[0], y = u[1], z = u[2];
  if (t == 0) {
    features(x, y, z, out);
  } else {
    float d[3][kNB];
    feature_derivs(x, y, z, d);
    // selects, not an indexed load: keeps d in registers
#pragma unroll
    for (int k = 0; k < kNB; ++k) out[k] = t == 1 ? d[0][k] : (t == 2 ? d[1][k] : d[2][k]);
  }
}

// The same row over the three emulator classes: entry 20 q + k is
// w_q phi_k, and its derivative rows carry d w_q / d u1 phi_k as well.
__device__ inline void feature_row_classes(const Geometry &g, const float *u, int t, float *out) {
  const float x = u[0], y = u[1], z = u[2];
  float phi[kNB], r[kNB], d[3][kNB];
  features(x, y, z, phi);
  feature_derivs(x, y, z, d);
#pragma unroll
  for (int k = 0; k < kNB; ++k)
    r[k] = t == 0 ? phi[k] : (t == 1 ? d[0][k] : (t == 2 ? d[1][k] : d[2][k]));
  float w[kMaxClasses], dw[kMaxClasses];
  class_weights(g, x, w, dw);
#pragma unroll
  for (int q = 0; q < kMaxClasses; ++q)
#pragma unroll
    for (int k = 0; k < kNB; ++k)
      out[kNB * q + k] = t == 1 ? fmaf(dw[q], phi[k], w[q] * r[k]) : w[q] * r[k];
}

// dJ/du_t (t = 1..3) from Phi-bar and d phi / d u_t (one emulator class).
__device__ inline float shape_gradient(const float *pb, const float *d) {
  float acc = 0.f;
#pragma unroll
  for (int k = 1; k < kNB; ++k) acc = fmaf(pb[k], d[k], acc);
  return acc;
}

// Adam's step number `step` (1, 2, ...): what all parameters share, and one
// parameter's update.
struct AdamStep {
  float step_size, rbc2;
};
__device__ inline AdamStep adam_step(const AdamCfg &c, int step) {
#pragma clang fp contract(off)
  const float bc1 = 1.f - powf(c.beta1, (float)step);
  const float bc2 = 1.f - powf(c.beta2, (float)step);
  return AdamStep{c.lr / bc1, 1.f / sqrtf(bc2)};
}
__device__ inline void adam_update(const AdamCfg &c, const AdamStep &s, float grad, float &m,
                                   float &v, float &u) {
#pragma clang fp contract(off)
  m = fmaf(c.beta1, m, (1.f - c.beta1) * grad);
  v = fmaf(c.beta2, v, (1.f - c.beta2) * grad * grad);
  const float denom = fmaf(sqrtf(v), s.rbc2, c.eps);
  u = fmaf(-s.step_size, m / denom, u);
}

// Makes the compiler treat x as a new value: computations from x after this
// point are not merged with the same computations before it (which would
// keep their results live across phases and raise register pressure).
template <typename T>
__device__ inline void opaque(T &x) {
  asm volatile("" : "+v"(x));
}

// Value of v in lane l (l wave uniform), through scalar registers.
__device__ inline double read_lane(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Orders a wave's LDS accesses so that lanes see each other's stores.
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sum over each aligned group of eight lanes, returned in all eight, by DPP
// lane moves (no LDS round trip): swap neighbours, swap pairs within a
// quad, then mirror within the half row, which pairs the group's two quads.
// The additions form the same tree in every lane, so all eight agree.
template <int CTRL>
__device__ inline float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ inline double dpp_mov(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
template <int CTRL>
__device__ inline int dpp_mov(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, false);
}
template <typename T>
__device__ inline T group8_sum(T v) {
  v += dpp_mov<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_mov<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_mov<0x141>(v);  // row_half_mirror
  return v;
}

__device__ inline int read_lane(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ inline float read_lane(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// Sum over the wave, the same value in every lane: eight-lane groups, then
// the row mirror pairs the two groups of each 16-lane row, then the four
// row sums are read through scalar registers and added in a fixed order.
template <typename T>
__device__ inline T wave_sum(T x) {
  x = group8_sum(x);
  x += dpp_mov<0x140>(x);  // row_mirror
  return (read_lane(x, 0) + read_lane(x, 16)) + (read_lane(x, 32) + read_lane(x, 48));
}

__device__ inline float wave_min(float x) {
  x = fminf(x, dpp_mov<0xB1>(x));
  x = fminf(x, dpp_mov<0x4E>(x));
  x = fminf(x, dpp_mov<0x141>(x));
  x = fminf(x, dpp_mov<0x140>(x));
  return fminf(fminf(read_lane(x, 0), read_lane(x, 16)), fminf(read_lane(x, 32), read_lane(x, 48)));
}

// Sum of NV per-lane doubles over one wave through LDS (no workgroup
// barrier: any single wave may call it).  scratch holds 8 x 64 doubles;
// out[0..NV) (LDS) is valid in every lane after the call.  Deterministic.
template <int NV>
__device__ inline void wave_sum_lds(const double (&acc)[NV], double *scratch, double *out,
                                    int lane) {
  const int tt = lane >> 3, part = lane & 7;
#pragma unroll
  for (int c = 0; c < (NV + 7) / 8; ++c) {
#pragma unroll
    for (int t = 0; t < 8; ++t) scratch[t * 64 + lane] = (8 * c + t < NV) ? acc[(8 * c + t) % NV] : 0.0;
    wave_lds_sync();
    const double *row = scratch + tt * 64 + 8 * part;
    double v = ((row[0] + row[1]) + (row[2] + row[3])) + ((row[4] + row[5]) + (row[6] + row[7]));
    v = group8_sum(v);
    if (part == 0 && 8 * c + tt < NV) out[8 * c + tt] = v;
    wave_lds_sync();
  }
}

// Sum of NV per-lane values over the workgroup through LDS: eight values at
// a time are widened to FP64 and transposed through scratch[wave][8][64]
// (one wave's region is 4 KB), each group of eight lanes adds one value's 64
// partials, then the waves' results are added in a fixed order.  out[0..NV)
// is valid for every thread after the call.  Deterministic.
template <int NW, int NV, typename T>
__device__ inline void block_sum_lds(const T (&acc)[NV], double *scratch, double *red,
                                     double *out, int lane, int wave) {
  double *sc = scratch + wave * 512;
  const int tt = lane >> 3, part = lane & 7;
#pragma unroll
  for (int c = 0; c < (NV + 7) / 8; ++c) {
    // FP32 partials are widened 8 at a time, so few doubles are live at once
#pragma unroll
    for (int t = 0; t < 8; ++t)
      sc[t * 64 + lane] = (8 * c + t < NV) ? (double)acc[(8 * c + t) % NV] : 0.0;
    wave_lds_sync();
    const double *row = sc + tt * 64 + 8 * part;
    double v = ((row[0] + row[1]) + (row[2] + row[3])) + ((row[4] + row[5]) + (row[6] + row[7]));
    v = group8_sum(v);
    if (part == 0) red[wave * 64 + 8 * c + tt] = v;
    wave_lds_sync();
  }
  __syncthreads();
  const int t = threadIdx.x;
  if (t < NV) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) s += red[w * 64 + t];
    out[t] = s;
  }
  __syncthreads();
}

// block_sum_lds for FP32 partials: eight values at a time go through
// scratch[wave][8][64] as FP32 (2 KB per wave; half the registers and LDS of
// widening first); each group of eight lanes adds one value's eight-lane
// runs in FP32 and the rest -- across the groups, then the waves -- in FP64,
// in a fixed order.  out[0..NV) is
// valid for every thread after the call.  Deterministic.
template <int NW, int NV>
__device__ inline void block_sum_lds_f32(const float (&acc)[NV], float *scratch, double *red,
                                         double *out, int lane, int wave) {
  float *sc = scratch + wave * 8 * 64;
  const int tt = lane >> 3, part = lane & 7;
#pragma unroll
  for (int c = 0; c < (NV + 7) / 8; ++c) {
#pragma unroll
    for (int t = 0; t < 8; ++t) sc[t * 64 + lane] = (8 * c + t < NV) ? acc[(8 * c + t) % NV] : 0.f;
    wave_lds_sync();
    const float4 x0 = *reinterpret_cast<const float4 *>(sc + tt * 64 + 8 * part);
    const float4 x1 = *reinterpret_cast<const float4 *>(sc + tt * 64 + 8 * part + 4);
    double v = (double)(((x0.x + x0.y) + (x0.z + x0.w)) + ((x1.x + x1.y) + (x1.z + x1.w)));
    v = group8_sum(v);
    if (part == 0) red[wave * 64 + 8 * c + tt] = v;
    wave_lds_sync();
  }
  __syncthreads();
  const int t = threadIdx.x;
  if (t < NV) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) s += red[w * 64 + t];
    out[t] = s;
  }
  __syncthreads();
}

// ---- Preparation of one spectrum by one workgroup, shared by k_prepare and
//      the one-shot passes: pixel weights, n_eff and the flux weight w of
//      Eq. 6 (a flux quantile, Section 3.3 "Setting spectral weighting
//      factors") -----------------------------------------------------------

// Order-preserving map of a float to an unsigned key.
__device__ inline uint32_t fkey(float f) {
  uint32_t b = __float_as_uint(f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ inline float funkey(uint32_t k) {
  uint32_t b = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
  return __uint_as_float(b);
}

// Key of a pixel left out of the selection (no finite flux maps to it).
constexpr uint32_t kNoKey = 0xffffffffu;

// Scratch of the preparation in LDS, 32-bit words: two sets of per-wave
// partial results, used in turn, so that one barrier serves each sum.
constexpr int kPrepScratch = 3 * 8;

// What the preparation finds out about one spectrum.
struct RowInfo {
  int n_eff;
  uint32_t any_bad;  // some obs or ivar is not finite
  float w;
};

// Reads the spectrum's row, thread t pixels t + i BLOCK (coalesced), into
// o and iv -- (0, 0) for a pixel without weight -- and finds its flux weight:
// the requested quantile q of the valid fluxes (linear interpolation between
// order statistics), rounded to the nearest power of two so that o/w and
// W w^2 are exact in floating point.  The objective does not depend on w.
//
// Only the power of two is needed, so the order statistics are bracketed
// instead of sorted out: counts of the valid fluxes below and up to the two
// ends of one power's interval (2^(b - 1/2), 2^(b + 1/2)), drawn in by 2^-12
// of their value, show that both order statistics next to the quantile, and
// with them q, lie inside it; then w = 2^b whatever q is.  b starts from the
// mean flux and moves by one towards the quantile, which takes one or two
// counts over registers (four operations per pixel) on a spectrum.  One count
// finds nonpositive order statistics, for which w is 1.  Where neither closes
// -- order statistics on both sides of an end or within 2^-12 of it, widely
// scattered fluxes -- q is formed from the order statistics themselves, found
// bit by bit by the same kind of counts over order-preserving keys (objective
// of 30,000 x 300 px of negative fluxes: 466 us by that search, 271 by the one
// count).
//
// Every thread of the workgroup gets the same RowInfo.  scratch: kPrepScratch
// words of LDS, free again after a barrier.
template <int BLOCK>
__device__ inline RowInfo prepare_row(const float *o_row, const float *i_row, int P, float quantile,
                                      uint32_t *scratch, float (&o)[kNPL], float (&iv)[kNPL]) {
  constexpr int NW = BLOCK / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int slot = 0;
  auto total = [&](int v) {  // sum over the workgroup
    uint32_t *red = scratch + 8 * slot;
    slot ^= 1;
    v = wave_sum(v);
    if (lane == 0) red[wave] = (uint32_t)v;
    __syncthreads();
    int t = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += (int)red[w];
    return __builtin_amdgcn_readfirstlane(t);
  };
  // f(i) for the thread's pixels, by groups that a short row leaves out (rows
  // of more than 128 threads have over 2,000 pixels): covariance of 3,000 x
  // 300 px 167 -> 158 us, objective of 30,000 x 512 px 304 -> 284
  auto pixels = [&](auto &&f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) f(i);
    if (BLOCK > 128 || P > 4 * BLOCK) {
#pragma unroll
      for (int i = 4; i < 9; ++i) f(i);
      if (BLOCK > 128 || P > 9 * BLOCK) {
#pragma unroll
        for (int i = 9; i < kNPL; ++i) f(i);
      }
    }
  };
  if constexpr (BLOCK == 128) {
#pragma unroll
    for (int i = 4; i < kNPL; ++i) {
      o[i] = INFINITY;
      iv[i] = 0.f;
    }
  }
  pixels([&](int i) {
    const int j = min(tid + i * BLOCK, P - 1);
    o[i] = o_row[j];
    iv[i] = i_row[j];
  });
  int n = 0;
  float sum = 0.f, fin = 0.f;  // fin: NaN once a value is not finite
  pixels([&](int i) {
    fin = fmaf(o[i], 0.f, fmaf(iv[i], 0.f, fin));
    const bool ok = isfinite(o[i]) && isfinite(iv[i]) && iv[i] > 0.f && tid + i * BLOCK < P;
    n += ok ? 1 : 0;
    sum += ok ? o[i] : 0.f;
    o[i] = ok ? o[i] : INFINITY;  // above every valid flux in the counts
    iv[i] = ok ? iv[i] : 0.f;
  });
  RowInfo r{0, 0, 1.f};
  sum = wave_sum(sum);
  if (lane == 0) scratch[16 + wave] = __float_as_uint(sum);
  n = total(n | (fin != fin ? 1 << 16 : 0));  // at most 8,704 pixels, 512 flags
  r.n_eff = n & 0xffff;
  r.any_bad = n >> 16 != 0 ? 1u : 0u;
  sum = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) sum += __uint_as_float(scratch[16 + w]);
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < kNPL; ++i) o[i] = iv[i] > 0.f ? o[i] : 0.f;
  };
  if (!(quantile > 0.f) || r.n_eff == 0) {
    clear();
    return r;
  }

  const float pos = quantile * (float)(r.n_eff - 1);
  const uint32_t k0 = (uint32_t)floorf(pos);
  const float frac = pos - (float)k0;
  const uint32_t k1 = frac > 0.f && k0 + 1 < (uint32_t)r.n_eff ? k0 + 1 : k0;
  float w = 1.f;
  bool found = false;
  {
    const float mean = sum / (float)r.n_eff;
    int b = 0, dir = 0;
    bool go = mean > 0.f && isfinite(mean) && k0 < (uint32_t)r.n_eff;
    if (go) b = __builtin_amdgcn_readfirstlane((int)rintf(log2f(mean)));
    for (int it = 0; it < 8 && go; ++it) {
      if (b < -100 || b > 100) break;
      const float lo = ldexpf(0.70728f, b), hi = ldexpf(1.41387f, b);
      int c_lo = 0, c_hi = 0;
      pixels([&](int i) {
        c_lo += o[i] < lo ? 1 : 0;
        c_hi += o[i] <= hi ? 1 : 0;
      });
      const uint32_t c = (uint32_t)total(c_lo | c_hi << 16);
      if ((c & 0xffffu) <= k0 && k1 < c >> 16) {
        w = exp2f((float)b);
        found = true;
        break;
      }
      const int step = k0 < (c & 0xffffu) ? -1 : 1;
      go = dir == 0 || step == dir;  // past the quantile: the ends part it
      dir = step;
      b += step;
    }
  }
  if (!found) {  // both order statistics nonpositive: so is q, and w stays 1
    int c = 0;
    pixels([&](int i) { c += o[i] <= 0.f ? 1 : 0; });
    found = k1 < (uint32_t)total(c);
  }
  if (!found) {
    // keys in place of the fluxes; the k0-th smallest is the largest value
    // that at most k0 keys are below
    uint32_t kth = 0;
#pragma unroll
    for (int i = 0; i < kNPL; ++i) o[i] = __uint_as_float(iv[i] > 0.f ? fkey(o[i]) : kNoKey);
#pragma unroll 1
    for (uint32_t bit = 0x80000000u; bit != 0; bit >>= 1) {
      const uint32_t t = kth | bit;
      int c = 0;
      pixels([&](int i) { c += __float_as_uint(o[i]) < t ? 1 : 0; });
      if ((uint32_t)total(c) <= k0) kth = t;
    }
    const float v0 = funkey(kth);
    float q = v0;
    if (k1 > k0) {
      // the next one: the same key if another pixel holds it, else the
      // smallest above it
      int c = 0;
      uint32_t m = kNoKey;
#pragma unroll
      for (int i = 0; i < kNPL; ++i) {
        const uint32_t key = __float_as_uint(o[i]);
        c += key <= kth ? 1 : 0;
        m = key > kth ? min(m, key) : m;
      }
#pragma unroll
      for (int s = 32; s > 0; s >>= 1) m = min(m, (uint32_t)__shfl_xor(m, s));
      if (lane == 0) scratch[16 + wave] = m;  // the mean's partials have been read
      const uint32_t upto = (uint32_t)total(c);
#pragma unroll
      for (int v = 0; v < NW; ++v) m = min(m, scratch[16 + v]);
      const float v1 = k1 < upto ? v0 : funkey(m);
      q = v0 + frac * (v1 - v0);
    }
    if (q > 0.f && isfinite(q)) w = exp2f(rintf(log2f(q)));
#pragma unroll
    for (int i = 0; i < kNPL; ++i) o[i] = funkey(__float_as_uint(o[i]));
  }
  if (!(w > 0.f) || !isfinite(w) || !isfinite(1.f / (w * w))) w = 1.f;
  r.w = w;
  clear();
  return r;
}

// ---- Continuum moments of one lane's pixels (Eq. 6).  Every fused
//      multiply-add is written out and none left to the compiler, so that
//      all kernels get the same bits -------------------------------------

// Sums over one lane of y_j T_l (l <= D), y_j T_D T_k (k = 1..D) and z_j T_n
// (n <= D), one abscissa at a time.
template <int ND>
struct MomentSums {
  float nu[ND], q[ND], rr[ND];  // q[0] unused
  __device__ inline void clear() {
#pragma unroll
    for (int k = 0; k < ND; ++k) nu[k] = q[k] = rr[k] = 0.f;
  }
  __device__ inline void add(float x, float y, float z) {
#pragma clang fp contract(off)
    const float x2 = x + x;
    float t[ND];  // T_0(x) .. T_D(x)
    t[0] = 1.f;
    t[1] = x;
#pragma unroll
    for (int l = 2; l < ND; ++l) t[l] = fmaf(x2, t[l - 1], -t[l - 2]);
    const float yd = y * t[ND - 1];
    nu[0] += y;
    rr[0] += z;
#pragma unroll
    for (int l = 1; l < ND; ++l) {
      nu[l] = fmaf(y, t[l], nu[l]);
      q[l] = fmaf(yd, t[l], q[l]);
      rr[l] = fmaf(z, t[l], rr[l]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
};

// The same sums by nodes: the pixels' W F''^2 and W F'' o are folded onto the
// nodes, 24 operations per pair of pixels against 2 x 47 (D = 10), and only
// the nodes go through the Chebyshev recurrence.
template <int ND>
__device__ inline void moments_by_nodes(MomentSums<ND> &s, float x_mid, float h,
                                        const float (&fpp)[kNPL], const float2 (&ow)[kNPL]) {
#pragma clang fp contract(off)
  float ye[kPairs + 1], yo[kPairs], ze[kPairs + 1], zo[kPairs];
  {
    const float wf = ow[kMid].y * fpp[kMid];
    const float y = wf * fpp[kMid], z = wf * ow[kMid].x;
#pragma unroll
    for (int c = 0; c <= kPairs; ++c) {
      ye[c] = y * kMomentNodes.e[c][0];
      ze[c] = z * kMomentNodes.e[c][0];
    }
#pragma unroll
    for (int c = 0; c < kPairs; ++c) yo[c] = zo[c] = 0.f;
  }
#pragma unroll
  for (int t = 1; t <= kMid; ++t) {
    const float wp = ow[kMid + t].y * fpp[kMid + t], wm = ow[kMid - t].y * fpp[kMid - t];
    const float yp = wp * fpp[kMid + t], ym = wm * fpp[kMid - t];
    const float zp = wp * ow[kMid + t].x, zm = wm * ow[kMid - t].x;
    const float ys = yp + ym, yd = yp - ym, zs = zp + zm, zd = zp - zm;
#pragma unroll
    for (int c = 0; c <= kPairs; ++c) {
      ye[c] = fmaf(kMomentNodes.e[c][t], ys, ye[c]);
      ze[c] = fmaf(kMomentNodes.e[c][t], zs, ze[c]);
    }
#pragma unroll
    for (int c = 0; c < kPairs; ++c) {
      yo[c] = fmaf(kMomentNodes.o[c][t], yd, yo[c]);
      zo[c] = fmaf(kMomentNodes.o[c][t], zd, zo[c]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  s.clear();
#pragma unroll
  for (int c = 0; c < kPairs; ++c) {
    const float dx = (float)kMomentNodes.tau[c] * h;
    s.add(x_mid + dx, ye[c] + yo[c], ze[c] + zo[c]);
    s.add(x_mid - dx, ye[c] - yo[c], ze[c] - zo[c]);
  }
  s.add(x_mid, ye[kPairs], ze[kPairs]);
}

// One lane's moments nu_0..nu_D, q_1..q_D, r_0..r_D in acc, by the nodes or
// over the pixels.  (Two kernels, not a branch: both forms in one kernel
// spilled 68 B per lane at 128 registers, either alone none.)
template <bool NODES, int ND>
__device__ inline void lane_moments(int j0, int P, const float (&fpp)[kNPL],
                                    const float2 (&ow)[kNPL], float (&acc)[3 * ND - 1]) {
#pragma clang fp contract(off)
  const float h = 2.f / (float)P;
  MomentSums<ND> s;
  if constexpr (NODES) {
    moments_by_nodes<ND>(s, fmaf((float)(j0 + kMid), h, -1.f), h, fpp, ow);
  } else {
    const float x0 = fmaf((float)j0, h, -1.f);
    s.clear();
#pragma unroll
    for (int i = 0; i < kNPL; ++i) {
      const float wf = ow[i].y * fpp[i];
      s.add(fmaf((float)i, h, x0), wf * fpp[i], wf * ow[i].x);
    }
  }
#pragma unroll
  for (int k = 0; k < ND; ++k) acc[k] = s.nu[k];
#pragma unroll
  for (int k = 1; k < ND; ++k) acc[ND - 1 + k] = s.q[k];
#pragma unroll
  for (int k = 0; k < ND; ++k) acc[2 * ND - 1 + k] = s.rr[k];
}

// Normal equations A b = r of the continuum (A_mn = (nu_{m+n} + nu_|m-n|)/2)
// from the moments nu_0..nu_D, q_1..q_D, r_0..r_D (nu_{D+k} = 2 q_k -
// nu_{D-k}), solved in FP64 by one wave, lane i holding row i.

// nu_0 .. nu_2D mirrored about index D (sNu[D + l] = sNu[D - l] = nu_l), so
// that row i reads nu_{i+n} and nu_{|i-n|} at fixed offsets from sNu + i.
template <int ND>
__device__ inline void mirror_moments(const double *sMom, double *sNu, int lane) {
  constexpr int D = ND - 1, NNU = 2 * ND - 1;
  const int l = min(lane, NNU - 1);
  const double lo = sMom[l], hi = sMom[l <= D ? l : 2 * D - l];
  const double nu = l <= D ? lo : fma(2.0, lo, -hi);
  if (lane < NNU) sNu[D + lane] = nu;
  if (lane >= 1 && lane <= D) sNu[D - lane] = nu;
}

// Gauss-Jordan on NC - ND right-hand sides without scaling the pivot rows:
// row k stays as it is and every other row loses its column-k entry; the
// solutions are rhs[c] / diag of row i, diag its own entry.  The pivots are
// those of the scaled form.  Returns whether all of them are positive and
// finite.
template <int ND, int NC>
__device__ inline bool eliminate(const double (&rows)[NC], int lane, double (&rhs)[NC - ND],
                                 double &diag) {
#pragma clang fp contract(off)
  double a[NC];  // a local copy: stays in registers
#pragma unroll
  for (int n = 0; n < NC; ++n) a[n] = rows[n];
  bool ok = true;
#pragma unroll
  for (int k = 0; k < ND; ++k) {
    double piv[NC];
#pragma unroll
    for (int n = k; n < NC; ++n) piv[n] = read_lane(a[n], k);
    ok = ok && (piv[k] > 0.0) && isfinite(piv[k]);
    // 1 / pivot: the hardware estimate and two Newton steps
    double rp = __builtin_amdgcn_rcp(piv[k]);
    rp = fma(rp, fma(-piv[k], rp, 1.0), rp);
    rp = fma(rp, fma(-piv[k], rp, 1.0), rp);
    const double f = lane == k ? 0.0 : a[k] * rp;
#pragma unroll
    for (int n = k + 1; n < NC; ++n) a[n] = fma(-f, piv[n], a[n]);
  }
  double dg = a[0];
#pragma unroll
  for (int n = 1; n < ND; ++n) dg = lane == n ? a[n] : dg;
  diag = dg;
#pragma unroll
  for (int c = 0; c < NC - ND; ++c) rhs[c] = a[ND + c];
  return ok;
}

// Solves for b and leaves the continuum in sBd as a power series in the pixel
// offset v = j - P/2 from the row's centre: x_j = h v with h = 2 / P, so
// C = sum_n m_n h^n v^n with m_n = sum_k b_k [x^n] T_k.  b goes through LDS to
// every lane of the wave, the coefficients m_n h^n back to LDS.  sNu: 3 D + 1
// doubles of scratch, left holding the mirrored moments; sBd: 32 doubles.
template <int ND>
__device__ inline bool solve_continuum(const double *sMom, double *sNu, double *sBd,
                                       const Geometry &g, int lane) {
#pragma clang fp contract(off)
  constexpr int D = ND - 1, NNU = 2 * ND - 1;
  mirror_moments<ND>(sMom, sNu, lane);
  // lanes past row D repeat row D; only rows 0..D are read or stored
  const bool own = lane < ND;
  double a[ND + 1];
  a[ND] = sMom[NNU + min(lane, ND - 1)];
  wave_lds_sync();
  {
    const double *nr = sNu + min(lane, ND - 1);
#pragma unroll
    for (int n = 0; n < ND; ++n) a[n] = 0.5 * (nr[D + n] + nr[D - n]);
  }
  double b[1], dg;
  const bool ok = eliminate<ND, ND + 1>(a, lane, b, dg);
  if (own) sBd[16 + lane] = ok ? b[0] / dg : 0.0;
  wave_lds_sync();
  double bk[ND];
#pragma unroll
  for (int k = 0; k < ND; ++k) bk[k] = sBd[16 + k];
  double mm[ND];
#pragma unroll
  for (int n = 0; n < ND; ++n) {
    double m = 0.0;
#pragma unroll
    for (int k = n; k < ND; k += 2) m = fma(bk[k], (double)kChebPow.c[k][n], m);
    mm[n] = m * g.hpow[n];
  }
  if (lane == 0) {
#pragma unroll
    for (int n = 0; n < ND; ++n) sBd[n] = mm[n];
  }
  return ok;
}

// Terms of a lane's local expansion.  Rows of more than 128 lanes have over
// 2,000 pixels: there the terms past the sixth order add at most 1e-10 of the
// continuum's largest value (the seventh derivative of a degree-10 polynomial
// by Markov's bound).
constexpr int expansion_terms(int block, int nd) { return block == 128 || nd < 7 ? nd : 7; }

// Taylor coefficients of t -> C(x_{j0 + kMid} + h t): the series in v shifted
// to v0 = j0 + kMid - P/2 by repeated synthetic division (FP64), for Horner in
// FP32 at t = i - kMid, |h t| <= 16 / P.
template <int ND, int NC>
__device__ inline void expand_continuum(const double *sBd, int j0, int P, float (&cf)[NC]) {
  double a[ND];
#pragma unroll
  for (int n = 0; n < ND; ++n) a[n] = sBd[n];
  const double v0 = (double)(j0 + kMid) - 0.5 * (double)P;
#pragma unroll
  for (int k = 0; k < ND - 1 && k < NC; ++k)
#pragma unroll
    for (int n = ND - 2; n >= k; --n) a[n] = fma(v0, a[n + 1], a[n]);
#pragma unroll
  for (int n = 0; n < NC; ++n) cf[n] = (float)a[n];
}

// Folds one quantity v_i of a lane's pixels onto the nodes: Y[2 c], Y[2 c + 1]
// at x_mid +- h tau_c, Y[6] at x_mid.
template <typename V>
__device__ inline void fold_nodes(V &&v, float (&Y)[kNodes]) {
#pragma clang fp contract(off)
  float e[kPairs + 1], o[kPairs];
  const float v0 = v(kMid);
#pragma unroll
  for (int c = 0; c <= kPairs; ++c) e[c] = v0 * kMomentNodes.e[c][0];
#pragma unroll
  for (int c = 0; c < kPairs; ++c) o[c] = 0.f;
#pragma unroll
  for (int t = 1; t <= kMid; ++t) {
    const float vp = v(kMid + t), vm = v(kMid - t);
    const float s = vp + vm, d = vp - vm;
#pragma unroll
    for (int c = 0; c <= kPairs; ++c) e[c] = fmaf(kMomentNodes.e[c][t], s, e[c]);
#pragma unroll
    for (int c = 0; c < kPairs; ++c) o[c] = fmaf(kMomentNodes.o[c][t], d, o[c]);
  }
#pragma unroll
  for (int c = 0; c < kPairs; ++c) {
    Y[2 * c] = e[c] + o[c];
    Y[2 * c + 1] = e[c] - o[c];
  }
  Y[kNodes - 1] = e[kPairs];
}

#endif  // __HIPCC__

}  // namespace lasp
