// Parameter covariance at the final point (Section 2.2 stage 9: linear
// error propagation Sigma = s^2 (J^T J)^{-1} with s^2 = chi2 / (n_eff - 5)).
//
// The residual r_j = sqrt(W_j) (o_j - C_j F''_j) depends on the five
// parameters u and on the continuum coefficients b.  The u-block of the
// inverse normal matrix is the inverse of the Schur complement
//   S = Ju^T Ju - Ju^T Jb (Jb^T Jb)^{-1} Jb^T Ju,
// so with Jb^T Jb = A (the continuum Gram matrix) and X = Jb^T Ju only 5x5
// and (D+1)x5 sums are needed.  The five columns dF''/du are formed in
// forward mode: dF''/du_t = G (x) dF'/du_t for t = 1..3 (dF'/du_t from the
// derivative rows of the interpolator contraction) and
// dF''/du_{4,5} = (dG/dmu, dG/dsigma) (x) F' times the chain factors.
// The kernel is an evaluation of its own: it also gives chi2, the model, the
// status and the model Jacobian d(C F'')/du at fixed continuum, from the same
// sums as the fused pass (chi2 and the status bit for bit).
//
// The Levenberg-Marquardt polish (the curvature step that the paper's Section
// 4.5, future improvements, proposes for the Adam stage) is the same
// evaluation in a loop.  S du = q with q = Ju^T W e (no continuum term:
// Jb^T W e = 0 at the least-squares continuum) are the Gauss-Newton normal
// equations of the residual with the continuum profiled out; a step solves
// (S + lambda diag(S)) du = q in FP64, and is kept when chi2 falls (lambda /
// 10) or dropped (lambda * 10), as in Marquardt's method.
#include "lasp_internal.h"

// Every fused multiply-add is written out, so that chi2 and the status are
// those of the fused pass in each mode.
#pragma clang fp contract(off)

namespace lasp {
namespace {

constexpr int kOffF = 16;

template <int V>
struct IntC {
  static constexpr int value = V;
};

// What a launch does: kOneShot prepares its spectra from obs and ivar itself;
// kPrepared takes them from s.ow; kLm too, and iterates.
constexpr int kOneShot = 0, kPrepared = 1, kLm = 2;

struct CovLayout {
  int ks;
  int k_off;   // floats: taps [n_arms][3][ks]
  int d_off;   // floats: columns dF''/du_{1..3} [3][kNPL * block], pixel order
  int x_off;   // bytes: doubles
  int bytes;
};

// Doubles behind x_off, after the reductions' [nwaves][64]: moments, Ju^T W Ju
// and q, X and work [D + 1][5], the mirrored moments, the power series,
// scalars, for D <= 10.
constexpr int kMomLen = 32, kJJLen = 24, kXLen = 56, kNuLen = 32, kBdLen = 32, kScalLen = 16;
constexpr int kCovLen = kMomLen + kJJLen + 2 * kXLen + kNuLen + kBdLen + kScalLen;
// The polish's: its state, then the feature rows [nb][4] as floats.
constexpr int kLmLen = 44;

// The staged row region (floats [0, k_off)) holds F' rows for the
// convolutions, then the reductions' scratch and rows on their way out.  With
// one arm and margins up to 64, four workgroups of 128 threads share a CU's
// LDS (covariance of 8,000 x 1,550 px 345 us, 407 with three) and two of 256.
__host__ __device__ constexpr CovLayout cov_layout(const Geometry &g, int nwaves, bool lm) {
  CovLayout L{};
  int cols = kOffF + (g.ldF > kNPL * g.block ? g.ldF : kNPL * g.block) + 32;
  L.ks = ((2 * g.M + 1 + 7) & ~7) + 8;
  L.k_off = (cols + 3) & ~3;
  L.d_off = (L.k_off + g.n_arms * 3 * L.ks + 3) & ~3;
  const int fl_end = L.d_off + 3 * kNPL * g.block;
  L.x_off = ((fl_end * 4) + 15) & ~15;
  L.bytes = L.x_off + 8 * (nwaves * 64 + kCovLen) + (lm ? 8 * kLmLen + 4 * 4 * g.nb : 0);
  return L;
}
constexpr int cov_bytes(int block) {
  Geometry g{};
  g.M = 64;
  g.n_arms = 1;
  g.block = block;
  g.nb = kNB;
  return cov_layout(g, block / 64, true).bytes;
}
static_assert(4 * cov_bytes(128) <= 160 * 1024 && 2 * cov_bytes(256) <= 160 * 1024,
              "workgroups that share a CU");

// 5x5 symmetric positive definite solve (Cholesky, FP64); false if not SPD.
__device__ inline bool chol5(double (&a)[kNP][kNP], double (&x)[kNP]) {
#pragma unroll
  for (int j = 0; j < kNP; ++j) {
    double d = a[j][j];
#pragma unroll
    for (int k = 0; k < j; ++k) d = fma(-a[j][k], a[j][k], d);
    if (!(d > 0.0) || !isfinite(d)) return false;
    const double l = sqrt(d);
    a[j][j] = l;
#pragma unroll
    for (int i = j + 1; i < kNP; ++i) {
      double v = a[i][j];
#pragma unroll
      for (int k = 0; k < j; ++k) v = fma(-a[i][k], a[j][k], v);
      a[i][j] = v / l;
    }
  }
#pragma unroll
  for (int i = 0; i < kNP; ++i) {
    double v = x[i];
#pragma unroll
    for (int k = 0; k < i; ++k) v = fma(-a[i][k], x[k], v);
    x[i] = v / a[i][i];
  }
#pragma unroll
  for (int i = kNP - 1; i >= 0; --i) {
    double v = x[i];
#pragma unroll
    for (int k = i + 1; k < kNP; ++k) v = fma(-a[k][i], x[k], v);
    x[i] = v / a[i][i];
  }
  return true;
}

// State of one spectrum's Levenberg-Marquardt iteration, in LDS.
struct LmState {
  double S[kNP * kNP], q[kNP];  // normal equations at cur
  double c0;                    // chi2 there (NaN: equations not positive definite)
  double lambda, step_inf;      // damping, max |du| of the trial step (NaN: no step)
  float cur[8], pt[8];          // kept point, evaluated point
  int next, done, limit;        // next: what lm_decide found
};
static_assert(sizeof(LmState) <= kLmLen * sizeof(double) && (kCovLen + kLmLen) % 2 == 0,
              "LM state fits its LDS, the feature rows are 16-byte aligned");

// After the evaluation number it: the iteration has ended, its trial step was
// dropped, or kept (the normal equations there are wanted).
constexpr int kLmEnd = 0, kLmDropped = 1, kLmKept = 2;

// chi2 at the evaluated point is c1 (normal equations positive definite if
// ok): keep or drop the trial step and test for the end.  One wave, all lanes
// alike; lane 0 writes.
__device__ inline void lm_decide(LmState &m, double c1, bool ok, int it, int last, int lane) {
  const double c0 = m.c0, dinf = m.step_inf;
  double lam = m.lambda;
  bool take, done = false;
  if (it == 0) {
    take = true;
    lam = 1e-3;
  } else if (isfinite(dinf) && isfinite(c1) && c1 < c0) {
    take = true;
    lam = fmax(lam * 0.1, 1e-15);
    done = (c0 - c1) <= kLmDropTol * c0 || dinf <= kLmStepTol;
  } else {
    take = false;
    lam *= 10.0;
    done = lam > kLmLambdaMax || (isfinite(dinf) && dinf <= kLmStepTol) || !isfinite(c0);
  }
  float u[kNP];
#pragma unroll
  for (int i = 0; i < kNP; ++i) u[i] = m.pt[i];
  wave_lds_sync();  // every lane has read the old state
  if (lane == 0) {
    m.lambda = lam;
    if (take) {
      m.c0 = ok ? c1 : NAN;
#pragma unroll
      for (int i = 0; i < kNP; ++i) m.cur[i] = u[i];
    }
    m.limit = !done && it == last;
    m.next = done || it == last ? kLmEnd : (take ? kLmKept : kLmDropped);
  }
}

// The next trial point from the normal equations at the kept one, or the end.
__device__ inline void lm_step(LmState &m, int lane) {
  const double lam = m.lambda;
  double a[kNP][kNP], x[kNP], q[kNP];
  double dmax = 0.0;
#pragma unroll
  for (int i = 0; i < kNP; ++i) {
    q[i] = m.q[i];
    x[i] = q[i];
#pragma unroll
    for (int j = 0; j < kNP; ++j) a[i][j] = m.S[i * kNP + j];
    dmax = fmax(dmax, a[i][i]);
  }
#pragma unroll
  for (int t = 0; t < kNP; ++t) a[t][t] = fma(lam, fmax(a[t][t], 1e-12 * dmax), a[t][t]);
  bool done = false;
  double step = 0.0;
  if (chol5(a, x)) {
    // predicted chi2 decrease of the Gauss-Newton model, du^T q: below the
    // tolerance there is nothing left to gain and the spectrum stops here
    double dec = 0.0;
#pragma unroll
    for (int t = 0; t < kNP; ++t) dec = fma(x[t], q[t], dec);
    done = dec < kLmDecreaseTol;
#pragma unroll
    for (int t = 0; t < kNP; ++t) {
      step = fmax(step, fabs(x[t]));
      if (lane == 0) m.pt[t] = (float)((double)m.cur[t] + x[t]);
    }
  } else {
    step = NAN;  // no step: the next evaluation raises lambda
#pragma unroll
    for (int t = 0; t < kNP; ++t)
      if (lane == 0) m.pt[t] = m.cur[t];
  }
  if (lane == 0) {
    m.step_inf = step;
    m.done = done ? 1 : 0;
  }
}

// Two waves per SIMD (two workgroups per CU, as the LDS allows).
//
// Bound by VALU issue: six convolutions, the moments, 15 + 5 products and 5
// columns against the Chebyshev polynomials per pixel.  The taps stop at the
// window's end, the continuum sums run over the lane's seven nodes (the five
// X columns fold 17 pixels onto them too), the continuum is a local expansion
// and chi2 comes from the same pass, so that no fused pass goes before.
// Measured at 16,384 x 3,900, covariance with its preparation and evaluation:
// 1.13 ms, against 1.31 + 0.25 + 0.45 ms as three kernels; after a fit, with
// the rows prepared, 1.07.  Jacobian of 509 x 7,800 px in three arms: 0.135
// ms against 0.33.
//
// kLm runs a spectrum's whole iteration in its workgroup: the F' rows at the
// trial point are formed here from the basis (in L2) -- the matrix cores'
// FP32 products are chains of fused multiply-adds over k in order, and the
// chain below is the same one bit for bit -- and nothing is launched, counted
// or waited for between iterations.  Row 0 and chi2 come first; the columns
// follow only where the point is kept and a step from it is still to be made.
// A plain fit, against six launches per iteration for all spectra: one of
// 1,550 px 375 -> 163 us (this kernel 126), 16,384 x 3,900 with the
// covariance 24.4 -> 7.9 ms (8.8 with every trial evaluated in full).
template <int BLOCK, int ND, int MODE, bool NODES>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(2))) void k_cov(
    Geometry g, State s, CovArgs ca) {
  constexpr int NW = BLOCK / 64;
  constexpr int NNU = 2 * ND - 1;
  constexpr int NMOM = NNU + ND;
  constexpr int NWIN = kNPL + kTB - 1;
  constexpr int NCOL = kNPL * BLOCK;  // stride of one staged column
  extern __shared__ __align__(16) unsigned char smem[];
  const CovLayout L = cov_layout(g, NW, MODE == kLm);
  float *sF = reinterpret_cast<float *>(smem);
  float *sK = sF + L.k_off;
  float *sD = sF + L.d_off;
  double *sRed = reinterpret_cast<double *>(smem + L.x_off);
  double *sMom = sRed + NW * 64;
  double *sJJ = sMom + kMomLen;   // JuJu packed [15], q [5]
  double *sX = sJJ + kJJLen;      // [ND][5]
  double *sW = sX + kXLen;        // work
  double *sNu = sW + kXLen;       // mirrored moments
  double *sBd = sNu + kNuLen;     // continuum power series
  double *sScal = sBd + kBdLen;   // [0] continuum solved, [1] chi2 (FP64 from the pixels up)
  int *sHa = reinterpret_cast<int *>(sScal + 4);        // [kMaxArms]
  float *sCs = reinterpret_cast<float *>(sScal + 8);    // [kMaxArms] chain factor for sigma
  static_assert(NMOM <= kMomLen && kNP * ND <= kXLen && 3 * ND - 2 <= kNuLen, "fits its LDS");
  LmState &lm = *reinterpret_cast<LmState *>(sScal + kScalLen);
  float4 *sPhi = reinterpret_cast<float4 *>(sScal + kScalLen + kLmLen);  // [nb]: phi and its derivatives

  const int spec = blockIdx.x;
  const int P = g.P, M = g.M;
  const bool multi = g.n_arms > 1;
  if (MODE == kLm && threadIdx.x < kNP) {
    const float u = s.u[(size_t)spec * kNP + threadIdx.x];
    lm.pt[threadIdx.x] = u;
    lm.cur[threadIdx.x] = u;
  }
  const int n4 = g.ldF / 4;
  float *fp = s.fp + (size_t)spec * s.fp_stride;

  // at most ca.last + 1 evaluations (kLm), else one
#pragma unroll 1
  for (int it = 0;; ++it) {
    // the thread's index is made anew in each evaluation: addresses and range
    // tests formed from it would be kept in registers over all of them
    int tid = threadIdx.x;
    if (MODE == kLm) opaque(tid);
    const int lane = tid & 63, wave = tid >> 6;
    const int j0 = tid * kNPL;
    const bool has_pix = j0 < P;
    const int wp0 = wave * 64 * kNPL;
    const int wp1 = min(wp0 + 64 * kNPL, P) - 1;
    int wa_lo = 0, wa_hi = 0;
    for (int a = 1; a < g.n_arms; ++a) {
      if (g.arm_start[a] <= wp0) wa_lo = a;
      if (g.arm_start[a] <= wp1) wa_hi = a;
    }
    __syncthreads();  // the point is set; the last evaluation's LDS is free
    const float *u = MODE == kLm ? lm.pt : s.u + (size_t)spec * kNP;

    // ---- taps G, dG/dmu, dG/dsigma per arm -------------------------------
    const double u4 = (double)u[3], u5 = (double)u[4];
    const double rv = g.rv_lo + (u4 + 1.0) * g.rv_half;
    const double sg = g.sg_lo + (u5 + 1.0) * g.sg_half;
    const double mu = rv * g.inv_scale;
    const float cmu = (float)(g.rv_half * g.inv_scale);
    if (wave == 0) {
      for (int a = 0; a < g.n_arms; ++a) {
        const double seff = g.bare ? sg : sqrt(sg * sg + g.arm_sig2[a]);
        double spx = seff * g.inv_scale;
        const bool fl = !(spx >= (double)kSigmaFloorPx);
        if (fl) spx = (double)kSigmaFloorPx;
        double hf = ceil(fabs(mu) + 5.0 * spx);
        if (!(hf <= (double)M)) hf = (double)M;
        const int H = (int)hf, T = 2 * H + 1;
        const double inv2s2 = 0.5 / (spx * spx);
        double gv[3], dv[3];
        double part = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const int idx = lane + 64 * k;
          double v = 0.0, d = 0.0;
          if (64 * k < T && idx < T) {
            d = (double)(idx - H) - mu;
            v = exp(-d * d * inv2s2);
          }
          gv[k] = v;
          dv[k] = d;
          part += v;
        }
        const double inv_sum = 1.0 / wave_sum(part);
        double s1 = 0.0, s2 = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          gv[k] *= inv_sum;
          s1 = fma(gv[k], dv[k], s1);
          s2 = fma(gv[k] * dv[k], dv[k], s2);
        }
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        const double r2 = 1.0 / (spx * spx), r3 = r2 / spx;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const int idx = lane + 64 * k;
          if (idx < L.ks) {
            const bool in = idx < T;
            sK[(a * 3 + 0) * L.ks + idx] = in ? (float)gv[k] : 0.f;
            sK[(a * 3 + 1) * L.ks + idx] = in ? (float)(gv[k] * (dv[k] - s1) * r2) : 0.f;
            sK[(a * 3 + 2) * L.ks + idx] = in ? (float)(gv[k] * fma(dv[k], dv[k], -s2) * r3) : 0.f;
          }
        }
        if (lane == 0) {
          sHa[a] = H;
          sCs[a] = fl ? 0.f : (float)(g.sg_half * g.inv_scale * (g.bare ? 1.0 : sg / seff));
        }
      }
    }
    if constexpr (MODE == kLm) {
      // ---- F' and its derivative rows at the trial point ------------------
      if (wave == NW - 1) {
        float pr[kNB * kMaxClasses];
        if (g.nb == kNB) {
          feature_row(u, lane & 3, pr);
#pragma unroll
          for (int k = 0; k < kNB; ++k)
            if (lane < 4) reinterpret_cast<float *>(sPhi)[4 * k + lane] = pr[k];
        } else {
          feature_row_classes(g, u, lane & 3, pr);
#pragma unroll
          for (int k = 0; k < kNB * kMaxClasses; ++k)
            if (lane < 4) reinterpret_cast<float *>(sPhi)[4 * k + lane] = pr[k];
        }
      }
      __syncthreads();
      const float4 *b4 = reinterpret_cast<const float4 *>(s.basis);
      auto form = [&](auto rows) {
#pragma unroll 1
        for (int q = tid; q < n4; q += BLOCK) {
          float4 r0 = make_float4(0.f, 0.f, 0.f, 0.f), r1 = r0, r2 = r0, r3 = r0;
          auto fold = [&](float4 &r, float p, const float4 &b) {
            r.x = fmaf(b.x, p, r.x);
            r.y = fmaf(b.y, p, r.y);
            r.z = fmaf(b.z, p, r.z);
            r.w = fmaf(b.w, p, r.w);
          };
          for (int k0 = 0; k0 < g.nb; k0 += kNB) {
#pragma unroll 10
            for (int k = 0; k < kNB; ++k) {
              const float4 b = b4[(size_t)(k0 + k) * n4 + q], p = sPhi[k0 + k];
              fold(r0, p.x, b);
              if constexpr (decltype(rows)::value == 4) {
                fold(r1, p.y, b);
                fold(r2, p.z, b);
                fold(r3, p.w, b);
              }
            }
          }
          // row 0 goes straight to its place; the derivative rows are read back
          // after a barrier (a row's last float4 by other threads, too)
          *reinterpret_cast<float4 *>(sF + kOffF + 4 * q) = r0;
          if constexpr (decltype(rows)::value == 4) {
            reinterpret_cast<float4 *>(fp + g.ldF)[q] = r1;
            reinterpret_cast<float4 *>(fp + 2 * g.ldF)[q] = r2;
            reinterpret_cast<float4 *>(fp + 3 * g.ldF)[q] = r3;
          }
        }
      };
      if (it < ca.last)
        form(IntC<4>{});
      else  // the last evaluation: chi2 only
        form(IntC<1>{});
    }

    // ---- forward-mode columns: F'' and dF''/du_t, one staged row at a time.
    //      Row 0 gives F'' and the mu, sigma columns (kept in registers); rows
    //      1..3 give the u1..u3 columns (kept in LDS) -------------------------
    float f[kNPL], d3[kNPL], d4[kNPL];
#pragma unroll
    for (int i = 0; i < kNPL; ++i) f[i] = d3[i] = d4[i] = 0.f;
    // the prepared data
    auto load_data = [&](float2 (&ow)[kNPL]) {
      const float2 *src = s.ow + (size_t)spec * kNPL * BLOCK + tid;  // lane-major, coalesced
#pragma unroll
      for (int i = 0; i < kNPL; ++i) ow[i] = src[i * BLOCK];
    };
    // continuum least squares, as in the fused pass; returns whether it is solved
    auto fit_continuum = [&](float2 (&ow)[kNPL]) {
#pragma unroll
      for (int i = 0; i < kNPL; ++i) {
        opaque(f[i]);
        opaque(ow[i]);
      }
      float acc[NMOM];
      int jb = j0;
      opaque(jb);  // the Chebyshev values formed here are not kept for the passes below
      lane_moments<NODES, ND>(jb, P, f, ow, acc);
      if constexpr (MODE == kLm && !NODES) {  // summed here, not, with every T_k held, where they are stored
#pragma unroll
        for (int k = 0; k < NMOM; ++k) opaque(acc[k]);
      }
      block_sum_lds_f32<NW, NMOM>(acc, sF, sRed, sMom, lane, wave);
      if (wave == 0) {
        const bool ok = solve_continuum<ND>(sMom, sNu, sBd, g, lane);
        if (lane == 0) sScal[0] = ok ? 1.0 : 0.0;
      }
      __syncthreads();
      return __builtin_amdgcn_readfirstlane((int)(sScal[0] != 0.0)) != 0;
    };
    // the staged row against NK rows of taps
    auto convolve = [&](auto nk, int H, int T, const float *K,
                        float (&acc)[decltype(nk)::value][kNPL]) {
      constexpr int NK = decltype(nk)::value;
#pragma unroll
      for (int q = 0; q < NK; ++q)
#pragma unroll
        for (int i = 0; i < kNPL; ++i) acc[q][i] = 0.f;
      for (int mb = 0; mb < T; mb += kTB) {
        const float *wsrc = sF + kOffF + j0 + M + H - mb - (kTB - 1);
        float w[NWIN];
#pragma unroll
        for (int q = 0; q < NWIN; ++q) w[q] = wsrc[q];
#pragma unroll
        for (int t = 0; t < kTB; ++t) {
          if (mb + t >= T) break;  // wave uniform
#pragma unroll
          for (int q = 0; q < NK; ++q) {
            const float gk = K[q * L.ks + mb + t];
#pragma unroll
            for (int i = 0; i < kNPL; ++i) acc[q][i] = fmaf(gk, w[i - t + kTB - 1], acc[q][i]);
          }
        }
      }
    };
    // F'' and the mu, sigma columns of arm a's pixels
    auto keep_first = [&](int a, int lo, int hi, const float (&acc)[3][kNPL]) {
      const float cs = sCs[a];
#pragma unroll
      for (int i = 0; i < kNPL; ++i)
        if (!multi || (j0 + i >= lo && j0 + i < hi)) {
          f[i] = acc[0][i];
          d3[i] = cmu * acc[1][i];
          d4[i] = cs * acc[2][i];
        }
    };
    float2 ow[kNPL];
    bool ok, kept = true;
    if constexpr (MODE == kLm) {
      for (int q = tid; q < kOffF; q += BLOCK) sF[q] = 0.f;
      for (int q = tid; q < 32; q += BLOCK) sF[kOffF + g.ldF + q] = 0.f;
      __syncthreads();
      for (int a = wa_lo; has_pix && a <= wa_hi; ++a) {
        const int H = __builtin_amdgcn_readfirstlane(sHa[a]), T = 2 * H + 1;
        const int lo = multi ? g.arm_start[a] : 0, hi = multi ? g.arm_start[a + 1] : P;
        float acc[3][kNPL];
        convolve(IntC<3>{}, H, T, sK + a * 3 * L.ks, acc);
        keep_first(a, lo, hi, acc);
      }
      // chi2 alone decides what becomes of the trial step: one that is
      // dropped, and the last one, need no derivatives
      __syncthreads();  // every read of the staged row is done: sF becomes scratch
      load_data(ow);
      ok = fit_continuum(ow);
      constexpr int NC = expansion_terms(BLOCK, ND);
      float cf[NC];
      int jb = j0;
      opaque(jb);
      expand_continuum<ND, NC>(sBd, jb, P, cf);
      double chi2 = 0.0;
#pragma unroll
      for (int i = 0; i < kNPL; ++i) {
        const float t = (float)(i - kMid);
        float C = cf[NC - 1];
#pragma unroll
        for (int k = NC - 2; k >= 0; --k) C = fmaf(C, t, cf[k]);
        const float e = fmaf(-C, f[i], ow[i].x);
        chi2 = fma((double)ow[i].y * (double)e, (double)e, chi2);
      }
      chi2 = wave_sum(chi2);
      if (lane == 0) sRed[wave * 64] = chi2;
      __syncthreads();
      if (wave == 0) {
        double c1 = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) c1 += sRed[w * 64];
        lm_decide(lm, c1, ok, it, ca.last, lane);
      }
      __syncthreads();
      const int next = __builtin_amdgcn_readfirstlane(lm.next);
      if (next == kLmEnd) break;  // at the latest after evaluation ca.last
      kept = next == kLmKept;
    }
    if (kept) {
      for (int r = MODE == kLm ? 1 : 0; r < 4; ++r) {
        {
          const float4 *src = reinterpret_cast<const float4 *>(fp + (size_t)r * g.ldF);
          // five named values: an array here would go to memory
          static_assert((kNPL * BLOCK / 4 + BLOCK - 1) / BLOCK == 5, "float4 of a row per thread");
          const int q0 = min(tid, n4 - 1), q1 = min(tid + BLOCK, n4 - 1),
                    q2 = min(tid + 2 * BLOCK, n4 - 1), q3 = min(tid + 3 * BLOCK, n4 - 1),
                    q4 = min(tid + 4 * BLOCK, n4 - 1);
          const float4 x0 = src[q0], x1 = src[q1], x2 = src[q2], x3 = src[q3], x4 = src[q4];
          __syncthreads();  // the previous row has been read
          // threads past the row store the last float4 again (the same value)
          float4 *dst = reinterpret_cast<float4 *>(sF + kOffF);
          dst[q0] = x0;
          dst[q1] = x1;
          dst[q2] = x2;
          dst[q3] = x3;
          dst[q4] = x4;
        }
        if (r == (MODE == kLm ? 1 : 0)) {
          for (int q = tid; q < kOffF; q += BLOCK) sF[q] = 0.f;
          for (int q = tid; q < 32; q += BLOCK) sF[kOffF + g.ldF + q] = 0.f;
        }
        __syncthreads();
        if (!has_pix && r > 0) {  // lanes past the row: columns that weigh nothing
#pragma unroll
          for (int i = 0; i < kNPL; ++i) sD[(r - 1) * NCOL + j0 + i] = 0.f;
        }
        for (int a = wa_lo; has_pix && a <= wa_hi; ++a) {
          const int H = __builtin_amdgcn_readfirstlane(sHa[a]), T = 2 * H + 1;
          const int lo = multi ? g.arm_start[a] : 0;
          const int hi = multi ? g.arm_start[a + 1] : P;
          const float *K = sK + a * 3 * L.ks;
          if (r == 0) {
            float acc[3][kNPL];
            convolve(IntC<3>{}, H, T, K, acc);
            keep_first(a, lo, hi, acc);
          } else {
            float acc[1][kNPL];
            convolve(IntC<1>{}, H, T, K, acc);
            // pixels past the last arm's end weigh nothing; they take zero
#pragma unroll
            for (int i = 0; i < kNPL; ++i)
              if (!multi || (j0 + i >= lo && j0 + i < hi) || j0 + i >= P)
                sD[(r - 1) * NCOL + j0 + i] = j0 + i < P ? acc[0][i] : 0.f;
          }
        }
      }
      __syncthreads();  // every read of the staged row is done: sF becomes scratch

      // ---- data and continuum (kLm has them) ------------------------------------
      [[maybe_unused]] RowInfo row{};
      if constexpr (MODE == kOneShot) {
        float o[kNPL], iv[kNPL];
        row = prepare_row<BLOCK>(ca.os.obs + (size_t)spec * P, ca.os.ivar + (size_t)spec * P, P,
                                 ca.os.quantile, reinterpret_cast<uint32_t *>(sRed), o, iv);
        const float inv_w = 1.f / row.w, w2 = row.w * row.w;
#pragma unroll
        for (int i = 0; i < kNPL; ++i) sF[tid + i * BLOCK] = o[i] * inv_w;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kNPL; ++i) ow[i].x = sF[j0 + i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kNPL; ++i) sF[tid + i * BLOCK] = iv[i] * w2;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kNPL; ++i) ow[i].y = sF[j0 + i];
        __syncthreads();
        if (tid == 0) {
          s.neff[spec] = row.n_eff;
          s.wscale[spec] = row.w;
        }
      } else if constexpr (MODE == kPrepared) {
        load_data(ow);
      }
      if constexpr (MODE != kLm) ok = fit_continuum(ow);

      // ---- one pass per pixel: continuum C, residual e, the residual Jacobian
      //      columns ju_t = C dF''/du_t (scaled in place: registers for mu and
      //      sigma, LDS for u1..u3), and Ju^T W Ju (15) and q = Ju^T W e (5),
      //      each lane in FP32, lanes and waves in FP64.  chi2 twice: as the
      //      fused pass forms it, for the caller, and in FP64 from the pixels up,
      //      for the covariance's scale and for the polish, which compares two
      //      of them to 1e-10 -------------------------------------------------
      const float wsc = MODE == kOneShot ? row.w : s.wscale[spec];
      {
        constexpr int NC = expansion_terms(BLOCK, ND);
        float cf[NC];
        int jb = j0;
        opaque(jb);
        expand_continuum<ND, NC>(sBd, jb, P, cf);
        float acc[20];
#pragma unroll
        for (int k = 0; k < 20; ++k) acc[k] = 0.f;
        float chi2_part = 0.f, cmin = INFINITY;
        [[maybe_unused]] double chi2_64 = 0.0;
#pragma unroll
        for (int i = 0; i < kNPL; ++i) {
          const float t = (float)(i - kMid);
          float C = cf[NC - 1];
#pragma unroll
          for (int k = NC - 2; k >= 0; --k) C = fmaf(C, t, cf[k]);
          const float e = fmaf(-C, f[i], ow[i].x);
          const float we = ow[i].y * e;
          if constexpr (MODE != kLm) {
            chi2_64 = fma((double)ow[i].y * (double)e, (double)e, chi2_64);
            chi2_part = fmaf(we, e, chi2_part);
            cmin = fminf(cmin, jb + i < P ? C : INFINITY);
            if (ca.model_out) sF[jb + i] = (C * f[i]) * wsc;
          }
          float dd[kNP];
#pragma unroll
          for (int t3 = 0; t3 < 3; ++t3) {
            const float v = sD[t3 * NCOL + jb + i] * C;
            sD[t3 * NCOL + jb + i] = v;
            dd[t3] = v;
          }
          d3[i] *= C;
          d4[i] *= C;
          dd[3] = d3[i];
          dd[4] = d4[i];
          int k = 0;
#pragma unroll
          for (int p = 0; p < kNP; ++p) {
            const float wd = ow[i].y * dd[p];
#pragma unroll
            for (int q = 0; q <= p; ++q) {
              acc[k] = fmaf(wd, dd[q], acc[k]);
              ++k;
            }
          }
#pragma unroll
          for (int p = 0; p < kNP; ++p) acc[15 + p] = fmaf(we, dd[p], acc[15 + p]);
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (MODE != kLm) {
          const double c64 = wave_sum(chi2_64);
          const double cs = wave_sum((double)chi2_part);
          const float cm = wave_min(cmin);
          if (lane == 0) {
            sRed[wave * 64 + 0] = cs;
            sRed[wave * 64 + 1] = (double)cm;
            sRed[wave * 64 + 2] = c64;
          }
          __syncthreads();
          if (tid == 0) {
            double c64 = 0.0;
#pragma unroll
            for (int w = 0; w < NW; ++w) c64 += sRed[w * 64 + 2];
            sScal[1] = c64;
          }
          if (tid == 0 && ca.set_status) {
            double cs = 0.0, cm = INFINITY;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
              cs += sRed[w * 64 + 0];
              cm = fmin(cm, sRed[w * 64 + 1]);
            }
            const int n_eff = MODE == kOneShot ? row.n_eff : s.neff[spec];
            s.chi2[spec] = cs;
            uint32_t st;
            if constexpr (MODE == kOneShot) {
              st = (row.any_bad ? kStNonfinite : 0u) | (n_eff <= kNP + g.nd ? kStNoData : 0u) |
                   box_bit(u);
              if (ca.os.J) ca.os.J[spec] = n_eff > 0 ? (float)(cs / (double)n_eff) : 0.f;
            } else {
              st = s.status[spec] & ~(kStSingular | kStContNonpos | kStSigmaFloor);
            }
            if (!ok) st |= kStSingular;
            if (!(cm > 0.0)) st |= kStContNonpos;
            for (int a = 0; a < g.n_arms; ++a) {
              const double seff = g.bare ? sg : sqrt(sg * sg + g.arm_sig2[a]);
              if (!(seff * g.inv_scale >= (double)kSigmaFloorPx)) st |= kStSigmaFloor;
            }
            s.status[spec] = st;
          }
          // rows leave in pixel order (the barrier above ends the pass)
          if (ca.model_out) {
            for (int j = tid; j < P; j += BLOCK) ca.model_out[(size_t)spec * P + j] = sF[j];
          }
          if (ca.out_jac) {
            float *o = ca.out_jac + (size_t)spec * kNP * P;
            for (int j = tid; j < P; j += BLOCK) {
#pragma unroll
              for (int t = 0; t < 3; ++t) o[(size_t)t * P + j] = sD[t * NCOL + j] * wsc;
            }
#pragma unroll
            for (int t = 3; t < kNP; ++t) {
              __syncthreads();
#pragma unroll
              for (int i = 0; i < kNPL; ++i) sF[j0 + i] = (t == 3 ? d3[i] : d4[i]) * wsc;
              __syncthreads();
              for (int j = tid; j < P; j += BLOCK) o[(size_t)t * P + j] = sF[j];
            }
          }
          if (!ca.out_cov) return;
          __syncthreads();  // sF becomes scratch again; the chi2 parts are read
        }
        block_sum_lds_f32<NW, 20>(acc, sF, sRed, sJJ, lane, wave);
      }
      // X[n][t] = Jb^T W Ju = sum W F'' T_n ju_t (Chebyshev T_n), FP32 per lane
      // and FP64 across lanes: one pass for the LDS columns u1..u3 and one for
      // the register columns mu, sigma (a pass that picked a register column by
      // a run-time index would make the compiler keep them in memory).
      {
#pragma unroll
        for (int i = 0; i < kNPL; ++i) f[i] = ow[i].y * f[i];
        const float h = 2.f / (float)P;
        auto xpass = [&](auto ncol, int t0, auto column) {
          constexpr int NCX = decltype(ncol)::value;
          int jb = j0;
          opaque(jb);
          float acc[NCX * ND];  // [column][n]
#pragma unroll
          for (int n = 0; n < NCX * ND; ++n) acc[n] = 0.f;
          auto add = [&](float x, const float (&v)[NCX]) {
            const float x2 = x + x;
#pragma unroll
            for (int c = 0; c < NCX; ++c) {
              acc[c * ND] += v[c];
              acc[c * ND + 1] = fmaf(v[c], x, acc[c * ND + 1]);
            }
            float tm = 1.f, tc = x;
#pragma unroll
            for (int n = 2; n < ND; ++n) {
              const float tn = fmaf(x2, tc, -tm);
#pragma unroll
              for (int c = 0; c < NCX; ++c) acc[c * ND + n] = fmaf(v[c], tn, acc[c * ND + n]);
              tm = tc;
              tc = tn;
            }
            __builtin_amdgcn_sched_barrier(0);
          };
          if constexpr (NODES) {
            float Y[NCX][kNodes];
#pragma unroll
            for (int c = 0; c < NCX; ++c) {
              fold_nodes([&](int i) { return f[i] * column(jb, c, i); }, Y[c]);
              __builtin_amdgcn_sched_barrier(0);
            }
            const float x_mid = fmaf((float)(jb + kMid), h, -1.f);
#pragma unroll
            for (int q = 0; q < kNodes; ++q) {
              float v[NCX];
#pragma unroll
              for (int c = 0; c < NCX; ++c) v[c] = Y[c][q];
              const float dx = q < 2 * kPairs ? (float)kMomentNodes.tau[q / 2 % kPairs] * h : 0.f;
              add(q % 2 == 0 && q < 2 * kPairs ? x_mid + dx : x_mid - dx, v);
            }
          } else {
#pragma unroll
            for (int i = 0; i < kNPL; ++i) {
              float v[NCX];
#pragma unroll
              for (int c = 0; c < NCX; ++c) v[c] = f[i] * column(jb, c, i);
              add(fmaf((float)(jb + i), h, -1.f), v);
            }
          }
          if constexpr (MODE == kLm && !NODES) {
#pragma unroll
            for (int n = 0; n < NCX * ND; ++n) opaque(acc[n]);
          }
          block_sum_lds_f32<NW, NCX * ND>(acc, sF, sRed, sW, lane, wave);
          if (tid < NCX * ND) sX[(tid % ND) * kNP + t0 + tid / ND] = sW[tid];
          __syncthreads();
        };
        xpass(IntC<3>{}, 0, [&](int jb, int c, int i) { return sD[c * NCOL + jb + i]; });
        xpass(IntC<2>{}, 3, [&](int, int c, int i) { return c == 0 ? d3[i] : d4[i]; });
      }

      // ---- wave 0: Y = A^{-1} X, S = JuJu - X^T Y --------------------------------
      if (wave == 0) {
        {
          double a[ND + kNP], y[kNP], dg;
          const double *nr = sNu + min(lane, ND - 1);
#pragma unroll
          for (int n = 0; n < ND; ++n) a[n] = 0.5 * (nr[ND - 1 + n] + nr[ND - 1 - n]);
#pragma unroll
          for (int t = 0; t < kNP; ++t) a[ND + t] = sX[min(lane, ND - 1) * kNP + t];
          ok = eliminate<ND, ND + kNP>(a, lane, y, dg) && ok;
          const double rd = 1.0 / dg;
          if (lane < ND) {
#pragma unroll
            for (int t = 0; t < kNP; ++t) sW[lane * kNP + t] = y[t] * rd;  // Y[n][t]
          }
        }
        wave_lds_sync();
        // lanes 0..4 own rows of S
        double sr[2 * kNP];
        const int r = lane < kNP ? lane : 0;
#pragma unroll
        for (int q = 0; q < kNP; ++q) {
          const int p = r > q ? r : q, qq = r > q ? q : r;
          sr[q] = sJJ[p * (p + 1) / 2 + qq];
          sr[kNP + q] = (r == q) ? 1.0 : 0.0;
        }
#pragma unroll
        for (int n = 0; n < ND; ++n) {
          const double x = sX[n * kNP + r];
#pragma unroll
          for (int q = 0; q < kNP; ++q) sr[q] = fma(-x, sW[n * kNP + q], sr[q]);
        }
        if constexpr (MODE == kLm) {
          if (lane < kNP) {
#pragma unroll
            for (int q = 0; q < kNP; ++q) lm.S[lane * kNP + q] = sr[q];
            lm.q[lane] = sJJ[15 + lane];
          }
        } else {
          // Sigma_u = s^2 S^{-1} by Gauss-Jordan on [S | I]
          double inv[kNP], dg;
          ok = eliminate<kNP, 2 * kNP>(sr, lane, inv, dg) && ok;
          const double rd = 1.0 / dg;
          const int n_eff = MODE == kOneShot ? row.n_eff : s.neff[spec];
          const double chi2 = sScal[1];
          const double s2 = n_eff > kNP ? chi2 / (double)(n_eff - kNP) : NAN;
          if (lane < kNP) {
            // physical units: Teff via dTeff = Teff ln10 dlog10Teff, the others by
            // the box half-widths
            const double lt = ca.lo[0] + 0.5 * ((double)u[0] + 1.0) * (ca.hi[0] - ca.lo[0]);
            double jd[kNP];
#pragma unroll
            for (int q = 0; q < kNP; ++q) jd[q] = 0.5 * (ca.hi[q] - ca.lo[q]);
            jd[0] *= exp10(lt) * kLn10;
            double jr = jd[0];
#pragma unroll
            for (int q = 1; q < kNP; ++q)
              if (q == lane) jr = jd[q];
#pragma unroll
            for (int q = 0; q < kNP; ++q) {
              const double v = ok ? s2 * (inv[q] * rd) * jr * jd[q] : NAN;
              ca.out_cov[((size_t)spec * kNP + lane) * kNP + q] = v;
            }
          }
          if (lane == 0 && !ok) s.status[spec] |= kStSingular;
        }
      }
      if constexpr (MODE != kLm) return;
    }
    if (wave == 0) {
      wave_lds_sync();
      lm_step(lm, lane);
    }
    __syncthreads();
    if (lm.done) break;
  }
  if (threadIdx.x < kNP) s.u[(size_t)spec * kNP + threadIdx.x] = lm.cur[threadIdx.x];
  if (threadIdx.x == 0 && lm.limit) s.status[spec] |= kStPolishLimit;
}

template <int BLOCK, int ND, int MODE, bool NODES>
hipError_t launch_cov_k(const Geometry &g, const State &s, const CovArgs &ca, hipStream_t st) {
  const CovLayout L = cov_layout(g, BLOCK / 64, MODE == kLm);
  auto k = k_cov<BLOCK, ND, MODE, NODES>;
  hipError_t e =
      hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, L.bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(g.B), dim3(BLOCK), L.bytes, st, g, s, ca);
  return hipGetLastError();
}

template <int BLOCK, int ND, int MODE>
hipError_t launch_cov_n(const Geometry &g, const State &s, const CovArgs &ca, hipStream_t st) {
  if constexpr (BLOCK == 128) {
    if (!moment_nodes_hold(ND, g.P)) return launch_cov_k<BLOCK, ND, MODE, false>(g, s, ca, st);
  }
  return launch_cov_k<BLOCK, ND, MODE, true>(g, s, ca, st);
}

template <int BLOCK, int MODE>
hipError_t launch_cov_b(const Geometry &g, const State &s, const CovArgs &ca, hipStream_t st) {
  switch (g.nd) {
    case 5: return launch_cov_n<BLOCK, 5, MODE>(g, s, ca, st);
    case 7: return launch_cov_n<BLOCK, 7, MODE>(g, s, ca, st);
    case 9: return launch_cov_n<BLOCK, 9, MODE>(g, s, ca, st);
    case 11: return launch_cov_n<BLOCK, 11, MODE>(g, s, ca, st);
    default: return hipErrorInvalidValue;
  }
}

template <int MODE>
hipError_t launch_cov_m(const Geometry &g, const State &s, const CovArgs &ca, hipStream_t st) {
  switch (g.block) {
    case 128: return launch_cov_b<128, MODE>(g, s, ca, st);
    case 256: return launch_cov_b<256, MODE>(g, s, ca, st);
    case 512: return launch_cov_b<512, MODE>(g, s, ca, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_cov_oneshot(const Geometry &g, const State &s, const CovArgs &ca,
                              hipStream_t st) {
  return launch_cov_m<kOneShot>(g, s, ca, st);
}

hipError_t launch_cov(const Geometry &g, const State &s, const CovArgs &ca, hipStream_t st) {
  return launch_cov_m<kPrepared>(g, s, ca, st);
}

hipError_t launch_lm(const Geometry &g, const State &s, const CovArgs &ca, hipStream_t st) {
  return launch_cov_m<kLm>(g, s, ca, st);
}

}  // namespace lasp
