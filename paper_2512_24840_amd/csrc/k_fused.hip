// Fused per-spectrum pass of one Adam step (Section 2.2, stages 4-8):
//   Eq. 5  Gaussian kernel G(mu, sigma) and F'' = F' (x) G, F' staged in LDS
//   Eq. 6  continuum by weighted least squares: moments of W F''^2 and
//          W F'' o against Chebyshev polynomials (per-lane FP32 sums over 17
//          pixels, FP64 across lanes), normal equations solved in FP64
//          (Gauss-Jordan, one lane per row)
//   Eq. 7  residual e = o - C F'' (C by Horner in a power series of the
//          pixel offset, re-centred on each lane's pixels);  Eq. 9
//          chi2 = sum W e^2 (per spectrum)
//   adjoint of J = chi2 / n_eff with the continuum at its least-squares
//          value (envelope theorem): g_j = -2 W e C / n_eff, the lag
//          correlation R(m) = sum_j g_j F'_{j-m+M} giving dJ/dmu and
//          dJ/dsigma, and the transposed convolution F-bar' that the
//          backward contraction turns into dJ/du_{1..3}.
//
// The continuum space {polynomials of degree <= D} is spanned here by
// Chebyshev polynomials: the least-squares fit, its residual, chi2 and the
// gradient are the same as with the paper's Legendre basis (only the
// coefficient vector differs), and T_m T_n = (T_{m+n} + T_{|m-n|}) / 2
// turns the Gram matrix into 2D + 1 moments.
//
// One workgroup owns one spectrum; lane l owns pixels [17 l, 17 l + 17) (an
// odd stride, so lanes hit distinct LDS banks).  Taps run in register blocks
// of 8 against a 24-value window.  The lag correlation takes g from
// registers, so the g-bar row the transposed convolution reads replaces F'
// in LDS once F' has been read for the last time.
#include <type_traits>

#include "lasp_internal.h"

// Every fused multiply-add below is written out: the compiler then forms none
// of its own, and the pass gives the same bits in each of its variants (a
// step, an evaluation of the returned point, a one-shot evaluation).
#pragma clang fp contract(off)

namespace lasp {
namespace {

constexpr int kOffF = 16;  // F' column c lives at sF[kOffF + c]

// What a launch of the pass does (see k_fused).
constexpr int kPass = 0, kOneShot = 1, kFit = 2;

// A block's taps (16-byte aligned in LDS, zeros past the window's end).
__device__ inline void load_taps(const float *k, float (&gk)[kTB]) {
  const float4 a = reinterpret_cast<const float4 *>(k)[0], b = reinterpret_cast<const float4 *>(k)[1];
  gk[0] = a.x;
  gk[1] = a.y;
  gk[2] = a.z;
  gk[3] = a.w;
  gk[4] = b.x;
  gk[5] = b.y;
  gk[6] = b.z;
  gk[7] = b.w;
}

// LDS of one workgroup.  Row region A holds, in turn, F' (column c at
// kOffF + c) until the lag correlation has read it, then the g-bar row
// (pixel j at 2M + j, j in [-2M, P + 2M + 32), zero outside [0, P)) for the
// transposed convolution, then F-bar' on its way out.  Scratch region B
// holds, in turn, the moments' reduction transposes, the lag correlation's
// per-wave transposes [NW][kTB][64] and wave 0's mu / sigma sums.
struct FusedLayout {
  int a_len;      // floats of region A
  int gb_base;    // 2M: g-bar pixel j at sF[gb_base + j]
  int b_off;      // float offset of region B
  int b_len;      // floats of region B
  int ks;         // taps buffer stride per arm
  int k_off;      // float offset of the taps
  int r_off;      // float offset of per-wave R(m) partials [NW][n_arms][ks]
  int rs_off;     // float offset of R(m) sums [n_arms][ks]
  int d_off;      // byte offset of the double scratch
  int fit_off;    // byte offset of the fit's state (FitLds)
  int bytes;
};

// What a whole fit in one workgroup keeps in LDS between its phases.
struct FitLds {
  float u[8], m[8], v[8];  // parameters and Adam moments
  float g45[2];            // dJ/du4, dJ/du5
  int t;                   // steps taken
  float part[8][kNB];      // Phi-bar's eight column parts
  float pb[kNB];           // Phi-bar
  AdamStep step;           // of the step under way
};

__host__ __device__ inline FusedLayout fused_layout(const Geometry &g, int nwaves, int nmom_pad) {
  FusedLayout L;
  const int f_len = kOffF + g.ldF + 32;
  const int g_len = g.P + 4 * g.M + 32;
  L.a_len = ((f_len > g_len ? f_len : g_len) + 3) & ~3;
  L.gb_base = 2 * g.M;
  const int mom = nwaves * 8 * 64;                          // FP32 moment transposes
  const int lag = nwaves * kTB * 64;
  const int musig = 2 * (8 * 64 + 8);                     // wave_sum_lds scratch + sums
  L.b_len = mom > lag ? mom : lag;
  if (L.b_len < musig) L.b_len = musig;
  L.b_off = L.a_len;
  L.ks = ((2 * g.M + 1 + 7) & ~7) + 8;
  L.k_off = L.b_off + L.b_len;
  L.r_off = L.k_off + g.n_arms * L.ks;
  L.rs_off = L.r_off + nwaves * g.n_arms * L.ks;
  int fl_end = L.rs_off + g.n_arms * L.ks;
  // the one-shot pass's row on its way into registers, from the start
  if (fl_end < kNPL * 64 * nwaves) fl_end = kNPL * 64 * nwaves;
  L.d_off = ((fl_end * 4) + 15) & ~15;
  // doubles: reduction scratch [nwaves][64], moments [nmom_pad], the
  // continuum's power series [32], scalars [32] (flag, per-arm H and sigma)
  L.fit_off = L.d_off + 8 * (nwaves * 64 + nmom_pad + 32 + 32);
  L.bytes = L.fit_off + (int)sizeof(FitLds);
  return L;
}

// set_status != 0: this pass evaluates the returned parameters; it replaces
// the evaluation bits (SINGULAR, CONT_NONPOS, SIGMA_FLOOR) of the spectrum's
// status with those of this pass.  0 (the passes of the Adam steps): the
// status is left alone, so a condition seen only on the way does not reach
// the result.
//
// Four waves per SIMD: the register budget is held to 128 per lane, so with
// the LDS above four 256-thread or two 512-thread workgroups share a CU.  No
// spills with one arm at 3,900 pixels, 52 bytes per lane with several arms;
// measured faster than three waves per SIMD, for both pixel counts.
//
// ONESHOT: the pass of an evaluation at given parameters (lasp_forward).  It
// prepares its spectrum itself: the row goes from obs and ivar through LDS
// into the lane's registers, and chi2, J, n_eff and the whole status are
// written from here.  A prepared (o/w, W w^2) array would be written once
// and read once, 69.6 KB of the 117 KB that one spectrum then moves, beside a
// launch of its own.  Measured at 65,536 x 3,900, preparation and pass:
// 1.48 ms, against 0.80 + 1.24 ms with k_prepare before it.
//
// FIT: many Adam steps of a spectrum in its workgroup, for groups too small to
// fill the chip, whose steps are bound by the latency of three kernels.  F' is
// formed here from the basis (in L2) and Phi-bar from F-bar' in LDS, by the
// same chains of fused multiply-adds as the contractions' matrix products, so
// a fit has the same bits on either path.  Its phases are latencies in a row
// (one workgroup per CU: taps come in vector loads, Phi-bar's first basis
// loads fly over two barriers, Adam's shared factors are formed beside another
// serial section), so it takes 256 registers a lane.  Per step, against three
// launches from a graph: one spectrum of 1,550 px 17.9 us (29.4), 100 of
// 3,900 px 21.7 us (44.0), 1,024 49.0 us (60.8).
//
// NODES: the continuum moments by nodes (moment_nodes_hold); always where the
// workgroup has more than 128 threads, as such rows have over 2,000 pixels.
template <int BLOCK, int ND, bool ADJ, bool MULTI, int MODE, bool NODES>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(MODE == kFit ? 2 : 4))) void k_fused(
    Geometry g, State s, float *model_out, int set_status, OneShot os, AdamCfg adam, int n_steps) {
  constexpr bool ONESHOT = MODE == kOneShot, FIT = MODE == kFit;
  constexpr int NW = BLOCK / 64;
  constexpr int NNU = 2 * ND - 1;  // nu_0 .. nu_{2D}
  constexpr int NMOM = NNU + ND;   // plus r_0 .. r_D
  constexpr int NWIN = kNPL + kTB - 1;
  constexpr bool kStep = ADJ && !ONESHOT;  // the pass of an Adam step: no status, no model
  extern __shared__ __align__(16) unsigned char smem[];
  const FusedLayout L = fused_layout(g, NW, NMOM);
  float *sF = reinterpret_cast<float *>(smem);  // region A
  float *sGb = sF + L.gb_base;  // sGb[j], j in [-2M, P + 2M + 32), once F' is read
  float *sB = sF + L.b_off;     // region B
  float *sK = sF + L.k_off;
  float *sRp = sF + L.r_off;
  float *sRs = sF + L.rs_off;
  double *sRed = reinterpret_cast<double *>(smem + L.d_off);
  double *sMom = sRed + NW * 64;
  double *sBd = sMom + NMOM;  // continuum power series m_n h^n
  double *sScal = sBd + 32;
  int *sHa = reinterpret_cast<int *>(sScal + 16);      // [kMaxArms]
  double *sSp = sScal + 24;                            // [kMaxArms]

  if ((int)blockIdx.x >= work_count(g, s)) return;  // past the active list
  const int spec = work_spec(s, blockIdx.x);
  if (ADJ && !slot_active(s, spec)) return;  // finished slot: no step
  const int P = g.P, M = g.M;
  FitLds &fl = *reinterpret_cast<FitLds *>(smem + L.fit_off);
  if constexpr (FIT) {
    if (threadIdx.x < kNP) {
      fl.u[threadIdx.x] = s.u[(size_t)spec * kNP + threadIdx.x];
      fl.m[threadIdx.x] = s.m[(size_t)spec * kNP + threadIdx.x];
      fl.v[threadIdx.x] = s.v[(size_t)spec * kNP + threadIdx.x];
    }
    if (threadIdx.x == 0) fl.t = s.t[spec];
    __syncthreads();
  }
#pragma unroll 1
  for (int it = 0;; ++it) {  // n_steps times (FIT), else once
    // the thread's index is made anew in each step of a fit: addresses and range
    // tests formed from it would be kept in registers over all of them
    int tid = threadIdx.x;
    if constexpr (FIT) opaque(tid);
    const int lane = tid & 63, wave = tid >> 6;
    const int j0 = tid * kNPL;           // first pixel (and basis column) of this lane
    float *sRt = sB + wave * (kTB * 64);
    // waves whose every lane has kNPL pixels in the row skip the per-pixel
    // range tests: wave-uniform branches
    const bool pix_inside = (__builtin_amdgcn_readfirstlane(wave) + 1) * 64 * kNPL <= g.P;
    auto branch = [](bool c, auto &&f) {
      if (c)
        f(std::true_type{});
      else
        f(std::false_type{});
    };
    const bool has_pix = j0 < P;
    const int jr = has_pix ? j0 : 0;     // window origin kept in range for idle lanes

    // ---- loads: the velocity and width first, then F' and the data, so that
    //      the F' stores below need not wait for the data ---------------------
    const float *u = FIT ? fl.u : s.u + (size_t)spec * kNP;
    const double u4 = (double)u[3];
    const double u5 = (double)u[4];
    // 17 * BLOCK >= ldF, so every thread stages at most five float4 of F'.
    constexpr int kStage = (kNPL * BLOCK / 4 + BLOCK - 1) / BLOCK;
    const int n4 = g.ldF / 4;
    const float4 *fsrc = reinterpret_cast<const float4 *>(s.fp + (size_t)spec * s.fp_stride);
    float4 fst[kStage];
    if constexpr (MODE == kPass) {
#pragma unroll
      for (int k = 0; k < kStage; ++k) fst[k] = fsrc[min(tid + k * BLOCK, n4 - 1)];
    }
    if constexpr (FIT) {
      // F' = Phi(u) B, a float4 of columns at a time: features in order, as the
      // forward contraction's products add them
      float phi[kNB];
      features(u[0], u[1], u[2], phi);
      const float4 *b4 = reinterpret_cast<const float4 *>(s.basis);
#pragma unroll 1
      for (int q = tid; q < n4; q += BLOCK) {
        float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int k = 0; k < kNB; ++k) {
          const float4 b = b4[k * n4 + q];
          r.x = fmaf(b.x, phi[k], r.x);
          r.y = fmaf(b.y, phi[k], r.y);
          r.z = fmaf(b.z, phi[k], r.z);
          r.w = fmaf(b.w, phi[k], r.w);
        }
        *reinterpret_cast<float4 *>(sF + kOffF + 4 * q) = r;
      }
    }
    float2 ow[kNPL];  // (o / w, W w^2)
    [[maybe_unused]] RowInfo row{};
    if constexpr (ONESHOT) {
      // the row in pixel order through region A, its two halves in turn; lane l
      // takes pixels [17 l, 17 l + 17) of each
      float o[kNPL], iv[kNPL];
      row = prepare_row<BLOCK>(os.obs + (size_t)spec * P, os.ivar + (size_t)spec * P, P, os.quantile,
                               reinterpret_cast<uint32_t *>(smem + L.d_off), o, iv);
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
      if (os.write_ow) {
        float2 *dst = s.ow + (size_t)spec * kNPL * BLOCK + tid;
#pragma unroll
        for (int i = 0; i < kNPL; ++i) dst[i * BLOCK] = ow[i];
      }
      if (tid == 0) {
        s.neff[spec] = row.n_eff;
        s.wscale[spec] = row.w;
      }
    } else {
      const float2 *src = s.ow + (size_t)spec * kNPL * BLOCK + tid;  // lane-major: coalesced
#pragma unroll
      for (int i = 0; i < kNPL; ++i) ow[i] = src[i * BLOCK];
    }
    if constexpr (!FIT) {
      // threads past the row store the last float4 again (the same value)
#pragma unroll
      for (int k = 0; k < kStage; ++k) {
        const int q = min(tid + k * BLOCK, n4 - 1);
        *reinterpret_cast<float4 *>(sF + kOffF + 4 * q) = ONESHOT ? fsrc[q] : fst[k];
      }
    }
    for (int q = tid; q < kOffF; q += BLOCK) sF[q] = 0.f;
    for (int q = tid; q < 32; q += BLOCK) sF[kOffF + g.ldF + q] = 0.f;
    for (int q = tid; q < NW * g.n_arms * L.ks; q += BLOCK) sRp[q] = 0.f;

    // ---- Eq. 5 kernel parameters: mu, sigma in pixels, H per arm (FP64) ----
    // Wave 0's serial sections (these taps, the continuum solve, dJ/dmu and
    // dJ/dsigma) run at raised wave priority: the other waves of the
    // workgroup wait on them, the waves of other workgroups do not.
    const double rv = g.rv_lo + (u4 + 1.0) * g.rv_half;
    const double sg = g.sg_lo + (u5 + 1.0) * g.sg_half;
    const double mu = rv * g.inv_scale;
    if (wave == 0) {
      __builtin_amdgcn_s_setprio(3);
      for (int a = 0; a < g.n_arms; ++a) {
        const double seff = g.bare ? sg : sqrt(sg * sg + g.arm_sig2[a]);
        double spx = seff * g.inv_scale;
        if (!(spx >= (double)kSigmaFloorPx)) spx = (double)kSigmaFloorPx;
        double hf = ceil(fabs(mu) + 5.0 * spx);
        if (!(hf <= (double)M)) hf = (double)M;  // also catches NaN
        const int H = (int)hf, T = 2 * H + 1;
        const double inv2s2 = 0.5 / (spx * spx);
        double gv[3];
        double part = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const int idx = lane + 64 * k;
          double v = 0.0;
          if (64 * k < T && idx < T) {  // first test is wave uniform
            const double d = (double)(idx - H) - mu;
            v = exp(-d * d * inv2s2);
          }
          gv[k] = v;
          part += v;
        }
        const double inv_sum = 1.0 / wave_sum(part);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const int idx = lane + 64 * k;
          if (idx < L.ks) sK[a * L.ks + idx] = (float)(gv[k] * inv_sum);
        }
        if (lane == 0) {
          sHa[a] = H;
          sSp[a] = spx;
        }
      }
    }
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();

    // ---- arms touched by this wave's output pixels (wave uniform) ---------
    constexpr bool multi = MULTI;  // several spectrograph arms
    const int wp0 = wave * 64 * kNPL;
    const int wp1 = min(wp0 + 64 * kNPL, P) - 1;
    int wa_lo = 0, wa_hi = 0;
    for (int a = 1; a < g.n_arms; ++a) {
      if (g.arm_start[a] <= wp0) wa_lo = a;
      if (g.arm_start[a] <= wp1) wa_hi = a;
    }

    // ---- Eq. 5: F''_j = sum_m G(m) F'_{j-m+M} ------------------------------
    float fpp[kNPL];
#pragma unroll
    for (int i = 0; i < kNPL; ++i) fpp[i] = 0.f;
    if (has_pix) {
      for (int a = wa_lo; a <= wa_hi; ++a) {
        const int H = __builtin_amdgcn_readfirstlane(sHa[a]), T = 2 * H + 1;
        const float *K = sK + a * L.ks;
        float acc[kNPL];
#pragma unroll
        for (int i = 0; i < kNPL; ++i) acc[i] = 0.f;
        for (int mb = 0; mb < T; mb += kTB) {
          const float *wsrc = sF + kOffF + j0 + M + H - mb - (kTB - 1);
          float w[NWIN];
#pragma unroll
          for (int q = 0; q < NWIN; ++q) w[q] = wsrc[q];
          float gk[kTB];
          load_taps(K + mb, gk);
#pragma unroll
          for (int t = 0; t < kTB; ++t) {
            if (mb + t >= T) break;  // wave uniform: no work on the block's padding
#pragma unroll
            for (int i = 0; i < kNPL; ++i) acc[i] = fmaf(gk[t], w[i - t + kTB - 1], acc[i]);
          }
        }
        if constexpr (!multi) {
#pragma unroll
          for (int i = 0; i < kNPL; ++i) fpp[i] = acc[i];
        } else {
          const int lo = g.arm_start[a], hi = g.arm_start[a + 1];
#pragma unroll
          for (int i = 0; i < kNPL; ++i)
            if (j0 + i >= lo && j0 + i < hi) fpp[i] = acc[i];
        }
      }
    }

    // ---- Eq. 6 moments: nu_l = sum W F''^2 T_l (l <= 2D), r_n = sum W F'' o T_n
    //      (n <= D), from T_0 .. T_D only: T_{D+k} = 2 T_D T_k - T_{D-k}, so
    //      nu_{D+k} = 2 q_k - nu_{D-k} with q_k = sum W F''^2 T_D T_k (k =
    //      1..D).  Each lane folds its 17 pixels onto seven nodes where
    //      those hold the polynomials (NODES) and sums in FP32, eight lanes' sums are added in
    //      FP32 on their way through LDS; the sums over those groups and the
    //      waves, the combination and the solve are FP64.
    {
#pragma unroll
      for (int i = 0; i < kNPL; ++i) {
        opaque(fpp[i]);
        opaque(ow[i]);
      }
      float acc[NMOM];
      lane_moments<NODES, ND>(j0, P, fpp, ow, acc);
      block_sum_lds_f32<NW, NMOM>(acc, sB, sRed, sMom, lane, wave);
    }

    // ---- normal equations A b = r (A_mn = (nu_{m+n} + nu_|m-n|)/2), solved
    //      in FP64 by Gauss-Jordan elimination, lane i holding row i.  sMom
    //      holds nu_0..nu_D, then q_1..q_D with nu_{D+k} = 2 q_k - nu_{D-k}.
    if (wave == 0) {
      __builtin_amdgcn_s_setprio(3);
      // sRed is free until the residual's chi2 sums
      const bool ok = solve_continuum<ND>(sMom, sRed, sBd, g, lane);
      if (lane == 0) sScal[0] = ok ? 1.0 : 0.0;
      __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();

    // ---- Eq. 7 residual, Eq. 9 chi2, adjoint seed g = dJ/dF'' ---------------
    const bool ok = __builtin_amdgcn_readfirstlane((int)(sScal[0] != 0.0)) != 0;
    const int n_eff = ONESHOT ? row.n_eff : s.neff[spec];
    const float gscale = n_eff > 0 ? -2.f / (float)n_eff : 0.f;
    [[maybe_unused]] const float wsc = ONESHOT ? row.w : s.wscale[spec];
    float gb[kNPL];
    float chi2_part = 0.f;  // this lane's 17 terms; lanes and waves add in FP64
    float cmin = INFINITY;
    {
      constexpr int NC = expansion_terms(BLOCK, ND);
      float cf[NC];
      expand_continuum<ND, NC>(sBd, j0, P, cf);
      auto residual = [&](auto inside) {
#pragma unroll
        for (int i = 0; i < kNPL; ++i) {
          const int j = j0 + i;
          const float t = (float)(i - kMid);
          float C = cf[NC - 1];
#pragma unroll
          for (int k = NC - 2; k >= 0; --k) C = fmaf(C, t, cf[k]);
          const float e = fmaf(-C, fpp[i], ow[i].x);
          const float we = ow[i].y * e;
          chi2_part = fmaf(we, e, chi2_part);
          gb[i] = (we * C) * gscale;
          if constexpr (!kStep) {
            if constexpr (decltype(inside)::value)
              cmin = fminf(cmin, C);
            else
              cmin = fminf(cmin, j < P ? C : INFINITY);
            if (model_out != nullptr) {
              if (j < P) model_out[(size_t)spec * P + j] = (C * fpp[i]) * wsc;
            }
          }
        }
      };
      // (the three-arm kernel keeps one copy of the loop: two copies there
      // moved its spills and measured slower)
      if constexpr (MULTI)
        residual(std::false_type{});
      else
        branch(pix_inside, residual);
      if (!ok) {
#pragma unroll
        for (int i = 0; i < kNPL; ++i) gb[i] = 0.f;
      }
    }
    if constexpr (!FIT) {  // the parameters that a fit returns get a pass of their own
      {
        const double cs = wave_sum((double)chi2_part);
        if (lane == 0) sRed[wave * 64 + 0] = cs;
        if constexpr (!kStep) {
          const float cm = wave_min(cmin);
          if (lane == 0) sRed[wave * 64 + 1] = (double)cm;
        }
      }
      __syncthreads();
      if (tid == 0) {
        double cs = 0.0, cm = INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          cs += sRed[w * 64 + 0];
          if constexpr (!kStep) cm = fmin(cm, sRed[w * 64 + 1]);
        }
        s.chi2[spec] = cs;
        if (!kStep && set_status) {
          uint32_t st;
          if constexpr (ONESHOT) {
            st = (row.any_bad ? kStNonfinite : 0u) | (n_eff <= kNP + g.nd ? kStNoData : 0u) |
                 box_bit(u);
            if (os.J) os.J[spec] = n_eff > 0 ? (float)(cs / (double)n_eff) : 0.f;
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
      }
    }
    if (!ADJ) return;

    // ---- lag correlation R_a(m) = sum_{j in arm a} g_j F'_{j-m+M} ----------
    if (wp0 < P) {
      for (int a = wa_lo; a <= wa_hi; ++a) {
        const int H = __builtin_amdgcn_readfirstlane(sHa[a]), T = 2 * H + 1;
        float gm[kNPL];
        if constexpr (!multi) {
          branch(pix_inside, [&](auto inside) {
#pragma unroll
            for (int i = 0; i < kNPL; ++i)
              gm[i] = (decltype(inside)::value || has_pix) ? gb[i] : 0.f;
          });
        } else {
          const int lo = g.arm_start[a], hi = g.arm_start[a + 1];
#pragma unroll
          for (int i = 0; i < kNPL; ++i)
            gm[i] = (has_pix && j0 + i >= lo && j0 + i < hi) ? gb[i] : 0.f;
        }
        for (int mb = 0; mb < T; mb += kTB) {
          const float *wsrc = sF + kOffF + jr + M + H - mb - (kTB - 1);
          float w[NWIN];
#pragma unroll
          for (int q = 0; q < NWIN; ++q) w[q] = wsrc[q];
          float r[kTB];
#pragma unroll
          for (int t = 0; t < kTB; ++t) {
            float acc = 0.f;
            if (mb + t < T) {  // wave uniform
#pragma unroll
              for (int i = 0; i < kNPL; ++i) acc = fmaf(gm[i], w[i - t + kTB - 1], acc);
            }
            r[t] = acc;
          }
          // wave-wide sums of the kTB partials: transpose through LDS, each
          // group of 8 lanes adds one tap's 64 partials (fixed order)
#pragma unroll
          for (int t = 0; t < kTB; ++t) sRt[t * 64 + lane] = r[t];
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          {
            const int tt = lane >> 3, part = lane & 7;
            const float4 x0 = *reinterpret_cast<const float4 *>(sRt + tt * 64 + 8 * part);
            const float4 x1 = *reinterpret_cast<const float4 *>(sRt + tt * 64 + 8 * part + 4);
            float v = ((x0.x + x0.y) + (x0.z + x0.w)) + ((x1.x + x1.y) + (x1.z + x1.w));
            v = group8_sum(v);
            if (part == 0) sRp[(wave * g.n_arms + a) * L.ks + mb + tt] = v;
          }
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
      }
    }
    __syncthreads();  // every read of F' is done: region A takes the g-bar row
    branch(pix_inside, [&](auto inside) {
#pragma unroll
      for (int i = 0; i < kNPL; ++i)
        if (decltype(inside)::value || j0 + i < P) sGb[j0 + i] = gb[i];
    });
    for (int q = tid; q < 2 * M; q += BLOCK) sGb[q - 2 * M] = 0.f;
    for (int q = tid; q < 2 * M + 32; q += BLOCK) sGb[P + q] = 0.f;
    for (int q = tid; q < g.n_arms * L.ks; q += BLOCK) {
      float acc = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) acc += sRp[w * g.n_arms * L.ks + q];
      sRs[q] = acc;
    }
    __syncthreads();

    // ---- dJ/dmu, dJ/dsigma per arm and the chain to u4, u5 (wave 0) -------
    if (wave == 0) {
      __builtin_amdgcn_s_setprio(3);
      double g4 = 0.0, g5 = 0.0;
      for (int a = 0; a < g.n_arms; ++a) {
        const int H = __builtin_amdgcn_readfirstlane(sHa[a]), T = 2 * H + 1;
        double s1 = 0, s2 = 0, rg = 0, rgd = 0, rgd2 = 0;
        for (int idx = lane; idx < T; idx += 64) {
          const double d = (double)(idx - H) - mu;
          const double G = (double)sK[a * L.ks + idx];
          const double R = (double)sRs[a * L.ks + idx];
          const double gd = G * d, rgv = R * G;
          s1 += gd;
          s2 = fma(gd, d, s2);
          rg += rgv;
          rgd = fma(rgv, d, rgd);
          rgd2 = fma(rgv * d, d, rgd2);
        }
        {
          // region B is free once the lag correlation is done
          const double part[5] = {s1, s2, rg, rgd, rgd2};
          double *tot = reinterpret_cast<double *>(sB) + 512;
          wave_sum_lds<5>(part, reinterpret_cast<double *>(sB), tot, lane);
          s1 = tot[0];
          s2 = tot[1];
          rg = tot[2];
          rgd = tot[3];
          rgd2 = tot[4];
        }
        const double sp = sSp[a];
        const double dmu = (rgd - s1 * rg) / (sp * sp);
        const double dsig = (rgd2 - s2 * rg) / (sp * sp * sp);
        g4 += dmu * g.rv_half * g.inv_scale;
        const double seff = g.bare ? sg : sqrt(sg * sg + g.arm_sig2[a]);
        const bool fl = !(seff * g.inv_scale >= (double)kSigmaFloorPx);
        const double dsdu = fl ? 0.0 : g.sg_half * g.inv_scale * (g.bare ? 1.0 : sg / seff);
        g5 += dsig * dsdu;
      }
      if (lane == 0) {
        float *g45 = FIT ? fl.g45 : s.g45 + (size_t)spec * 2;
        g45[0] = ok ? (float)g4 : 0.f;
        g45[1] = ok ? (float)g5 : 0.f;
      }
      __builtin_amdgcn_s_setprio(0);
    }

    if (FIT && wave == NW - 1) {  // beside wave 0's section above
      const AdamStep as = adam_step(adam, fl.t + 1);
      if (lane == 0) fl.step = as;
    }

    // ---- transposed convolution F-bar'_c = sum_m G(m) g_{c+m-M} ------------
    const int c0 = j0;
    float fb[kNPL];
#pragma unroll
    for (int i = 0; i < kNPL; ++i) fb[i] = 0.f;
    if (c0 < g.Pe) {
      // arms whose pixels the columns of this wave can reach (wave uniform)
      int ta_lo = 0, ta_hi = 0;
      if constexpr (multi) {
        const int jlo = wave * 64 * kNPL - 2 * M;
        const int jhi = (wave + 1) * 64 * kNPL - 1;
        for (int a = 1; a < g.n_arms; ++a) {
          if (g.arm_start[a] <= jlo) ta_lo = a;
          if (g.arm_start[a] <= jhi) ta_hi = a;
        }
      }
      for (int a = ta_lo; a <= ta_hi; ++a) {
        const int H = __builtin_amdgcn_readfirstlane(sHa[a]), T = 2 * H + 1;
        const float *K = sK + a * L.ks;
        const int lo = multi ? g.arm_start[a] : 0;
        const int hi = multi ? g.arm_start[a + 1] : P;
        for (int mb = 0; mb < T; mb += kTB) {
          const int base = c0 - H + mb - M;
          float w[NWIN];
#pragma unroll
          for (int q = 0; q < NWIN; ++q) w[q] = sGb[base + q];
          if constexpr (multi) {
#pragma unroll
            for (int q = 0; q < NWIN; ++q) w[q] = (base + q >= lo && base + q < hi) ? w[q] : 0.f;
          }
          float gk[kTB];
          load_taps(K + mb, gk);
#pragma unroll
          for (int t = 0; t < kTB; ++t) {
            if (mb + t >= T) break;  // wave uniform
#pragma unroll
            for (int i = 0; i < kNPL; ++i) fb[i] = fmaf(gk[t], w[i + t], fb[i]);
          }
        }
      }
    }
    // Phi-bar's first loads of the basis (FIT), in flight over the two barriers.
    // Rows 0-15: a wave's column parts side by side, kAhead blocks of 16 columns
    // each; four neighbouring lanes read a row's 64 bytes (rows across
    // neighbouring lanes would put 16 cache lines in each quarter of a load).
    // Rows 16-19: eight lanes read a row's 128 bytes of a stage of 32 columns;
    // an odd last 16 columns belong to places 0-3 alone.
    constexpr int kSeg = 8 / NW, kAhead = 16 / kSeg, kPair = NW < 4 ? 4 / NW : 1, kStages = 8;
    const int per = g.ldF / 8, n16 = per / 16;
    const int r16 = lane >> 2, kq = lane & 3, f8 = lane & 7;
    const int n_st = f8 < 4 ? (n16 + 1) / 2 : n16 / 2;      // stages of this place
    const int col8 = n_st > 0 ? 4 * f8 : 0;                 // none: read what is there
    const float *b16 = s.basis + (size_t)r16 * g.ldF + wave * per + 4 * kq;
    const int part8 = 2 * min(wave, 3) + (lane >> 5);       // + 2 NW per further pair
    const float *b4row = s.basis + (size_t)(16 + ((lane >> 3) & 3)) * g.ldF + part8 * per + col8;
    float4 y[FIT ? kAhead : 1][FIT ? kSeg : 1], y4[FIT ? kPair : 1][FIT ? kStages : 1];
    auto fetch16 = [&](float4 (&x)[FIT ? kAhead : 1][FIT ? kSeg : 1], int b0) {
#pragma unroll
      for (int i = 0; i < kAhead; ++i)
#pragma unroll
        for (int q = 0; q < kSeg; ++q)
          x[i][q] = *reinterpret_cast<const float4 *>(b16 + NW * q * per + 16 * min(b0 + i, n16 - 1));
    };
    auto fetch4 = [&](int st0) {
#pragma unroll
      for (int p = 0; p < kPair; ++p)
#pragma unroll
        for (int i = 0; i < kStages; ++i)
          y4[p][i] = *reinterpret_cast<const float4 *>(b4row + 2 * NW * p * per +
                                                       32 * min(st0 + i, max(n_st - 1, 0)));
    };
    if constexpr (FIT) {
      fetch16(y, 0);
    }
    __syncthreads();  // every read of the g-bar row is done: region A takes F-bar'
#pragma unroll
    for (int i = 0; i < kNPL; ++i)
      if (c0 + i < g.ldF) sF[kOffF + c0 + i] = (c0 + i < g.Pe) ? fb[i] : 0.f;
    __syncthreads();
    if constexpr (!FIT) {
      float4 *dst = reinterpret_cast<float4 *>(s.fbar + (size_t)spec * g.ldF);
      for (int q = tid; q < g.ldF / 4; q += BLOCK)
        dst[q] = *reinterpret_cast<const float4 *>(sF + kOffF + 4 * q);
      return;
    } else {
      // ---- Phi-bar = F-bar' B^T in the adjoint contraction's order: eight
      //      column parts; rows 0-15 over the float4 at one place of every 16
      //      columns, rows 16-19 of every 32 ------------------------------------
      const float *sFb = sF + kOffF;
      auto chain = [](float &acc, const float4 &x, const float4 &b) {
        acc = fmaf(x.x, b.x, acc);
        acc = fmaf(x.y, b.y, acc);
        acc = fmaf(x.z, b.z, acc);
        acc = fmaf(x.w, b.w, acc);
      };
      {
        const float *fa = sFb + wave * per + 4 * kq;
        float acc[kSeg];
#pragma unroll
        for (int q = 0; q < kSeg; ++q) acc[q] = 0.f;
        auto use = [&](const float4 (&x)[kAhead][kSeg], int b0) {
#pragma unroll
          for (int i = 0; i < kAhead; ++i) {
            if (b0 + i >= n16) break;  // uniform
#pragma unroll
            for (int q = 0; q < kSeg; ++q)
              chain(acc[q], *reinterpret_cast<const float4 *>(fa + NW * q * per + 16 * (b0 + i)), x[i][q]);
          }
        };
        float4 z[kAhead][kSeg];
#pragma unroll 1
        for (int b0 = 0; b0 < n16; b0 += 2 * kAhead) {
          fetch16(z, b0 + kAhead);
          use(y, b0);
          fetch16(y, b0 + 2 * kAhead);
          use(z, b0 + kAhead);
        }
#pragma unroll
        for (int q = 0; q < kSeg; ++q) {
          acc[q] += dpp_mov<0xB1>(acc[q]);  // quad_perm [1, 0, 3, 2]
          acc[q] += dpp_mov<0x4E>(acc[q]);  // quad_perm [2, 3, 0, 1]
          if (kq == 0) fl.part[wave + NW * q][r16] = acc[q];
        }
      }
      if (wave < 4) {
        fetch4(0);
        float acc[kPair];
#pragma unroll
        for (int p = 0; p < kPair; ++p) acc[p] = 0.f;
#pragma unroll 1
        for (int st0 = 0;;) {
#pragma unroll
          for (int i = 0; i < kStages; ++i)
#pragma unroll
            for (int p = 0; p < kPair; ++p) {
              const int st = min(st0 + i, max(n_st - 1, 0));
              float4 x = *reinterpret_cast<const float4 *>(sFb + (part8 + 2 * NW * p) * per + col8 + 32 * st);
              if (st0 + i >= n_st) x = make_float4(0.f, 0.f, 0.f, 0.f);
              chain(acc[p], x, y4[p][i]);
            }
          st0 += kStages;
          if (st0 >= (n16 + 1) / 2) break;  // uniform
          fetch4(st0);
        }
#pragma unroll
        for (int p = 0; p < kPair; ++p) {
          acc[p] = group8_sum(acc[p]);
          if (f8 == 0) fl.part[part8 + 2 * NW * p][16 + ((lane >> 3) & 3)] = acc[p];
        }
      }
      __syncthreads();
      if (wave == 0) {
        // ---- gradient and Adam step, lane a parameter a ----------------------
        if (lane < kNB) {
          float v = fl.part[0][lane];
#pragma unroll
          for (int w = 1; w < 8; ++w) v += fl.part[w][lane];
          fl.pb[lane] = v;
        }
        wave_lds_sync();
        const int a = min(lane, kNP - 1);
        float dr[kNB];
        feature_row(u, min(a, 2) + 1, dr);
        const float shape = shape_gradient(fl.pb, dr);
        const float grad = a < 3 ? shape : fl.g45[a - 3 < 0 ? 0 : a - 3];
        const int step = fl.t + 1;
        const AdamStep as = fl.step;
        float un = fl.u[a], mn = fl.m[a], vn = fl.v[a];
        adam_update(adam, as, grad, mn, vn, un);
        wave_lds_sync();
        if (lane < kNP) {
          fl.u[lane] = un;
          fl.m[lane] = mn;
          fl.v[lane] = vn;
        }
        if (lane == 0) fl.t = step;
      }
      __syncthreads();
      if (it + 1 >= n_steps) break;
    }
  }
  if (threadIdx.x < kNP) {
    s.u[(size_t)spec * kNP + threadIdx.x] = fl.u[threadIdx.x];
    s.m[(size_t)spec * kNP + threadIdx.x] = fl.m[threadIdx.x];
    s.v[(size_t)spec * kNP + threadIdx.x] = fl.v[threadIdx.x];
  }
  if (threadIdx.x == 0) s.t[spec] = fl.t;
}

// Arguments of a launch of any mode.
struct PassArgs {
  int adjoint;
  float *model_out;
  int set_status;
  OneShot os;
  AdamCfg adam;
  int n_steps;
};

template <int BLOCK, int ND, bool ADJ, bool MULTI, int MODE, bool NODES>
hipError_t launch_fused_k(const Geometry &g, const State &s, const PassArgs &a, hipStream_t st) {
  const FusedLayout L = fused_layout(g, BLOCK / 64, 3 * ND - 1);
  auto k = k_fused<BLOCK, ND, ADJ, MULTI, MODE, NODES>;
  hipError_t e =
      hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, L.bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(g.B), dim3(BLOCK), L.bytes, st, g, s, a.model_out, a.set_status, a.os,
                     a.adam, a.n_steps);
  return hipGetLastError();
}

template <int BLOCK, int ND, int MODE, bool NODES>
hipError_t launch_fused_t(const Geometry &g, const State &s, const PassArgs &a, hipStream_t st) {
  const bool multi = g.n_arms > 1;
  if (MODE == kFit || a.adjoint)
    return multi ? launch_fused_k<BLOCK, ND, true, true, MODE, NODES>(g, s, a, st)
                 : launch_fused_k<BLOCK, ND, true, false, MODE, NODES>(g, s, a, st);
  if constexpr (MODE != kFit)
    return multi ? launch_fused_k<BLOCK, ND, false, true, MODE, NODES>(g, s, a, st)
                 : launch_fused_k<BLOCK, ND, false, false, MODE, NODES>(g, s, a, st);
  return hipErrorInvalidValue;
}

template <int BLOCK, int ND, int MODE>
hipError_t launch_fused_n(const Geometry &g, const State &s, const PassArgs &a, hipStream_t st) {
  if constexpr (BLOCK == 128) {
    if (!moment_nodes_hold(ND, g.P)) return launch_fused_t<BLOCK, ND, MODE, false>(g, s, a, st);
  }
  return launch_fused_t<BLOCK, ND, MODE, true>(g, s, a, st);
}

template <int BLOCK, int MODE>
hipError_t launch_fused_b(const Geometry &g, const State &s, const PassArgs &a, hipStream_t st) {
  switch (g.nd) {
    case 5: return launch_fused_n<BLOCK, 5, MODE>(g, s, a, st);
    case 7: return launch_fused_n<BLOCK, 7, MODE>(g, s, a, st);
    case 9: return launch_fused_n<BLOCK, 9, MODE>(g, s, a, st);
    case 11: return launch_fused_n<BLOCK, 11, MODE>(g, s, a, st);
    default: return hipErrorInvalidValue;
  }
}

template <int MODE>
hipError_t launch_fused_m(const Geometry &g, const State &s, const PassArgs &a, hipStream_t st) {
  switch (g.block) {
    case 128: return launch_fused_b<128, MODE>(g, s, a, st);
    case 256: return launch_fused_b<256, MODE>(g, s, a, st);
    case 512: return launch_fused_b<512, MODE>(g, s, a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

bool fused_supported(int block, int nd) {
  return (block == 128 || block == 256 || block == 512) &&
         (nd == 5 || nd == 7 || nd == 9 || nd == 11);
}

size_t fused_smem_bytes(const Geometry &g) {
  return (size_t)fused_layout(g, g.block / 64, 3 * g.nd - 1).bytes;
}

hipError_t launch_fused(const Geometry &g, const State &s, int adjoint, float *model_out,
                        int set_status, hipStream_t st) {
  return launch_fused_m<kPass>(g, s, PassArgs{adjoint, model_out, set_status, {}, {}, 0}, st);
}

hipError_t launch_fused_oneshot(const Geometry &g, const State &s, int adjoint, float *model_out,
                                const OneShot &os, hipStream_t st) {
  return launch_fused_m<kOneShot>(g, s, PassArgs{adjoint, model_out, 1, os, {}, 0}, st);
}

hipError_t launch_fit(const Geometry &g, const State &s, const AdamCfg &adam, int n_steps,
                      hipStream_t st) {
  return launch_fused_m<kFit>(g, s, PassArgs{1, nullptr, 0, {}, adam, n_steps}, st);
}

}  // namespace lasp
