// Clean outlier mask (Section 2.2, step 6: the three-step clipping of the
// Clean strategy), per spectrum, from the residual eps = o - m against the
// current model m:
//   B  |eps_j| - f G_j > k sigma, k = 3 relaxed to 4, 5, 7 while more than
//      3 % of the valid pixels would be clipped;
//   C  a neighbour of a B outlier with |eps| - f G > 2 sigma;
//   D  a neighbour j' of an outlier j with eps_j eps_j' > 0,
//      |eps_j'| <= |eps_j| and |eps_j'| - f G_j' > sigma', repeated until it
//      does not change (at most 20 passes);
// with G_j = max |m_j - m_{j+-1}| (the flux gradient), sigma the sample
// standard deviation of eps over the valid pixels and sigma' over those
// kept by B and C.  Decisions in FP64.  Only pixels with positive finite
// weight are tested or seed a neighbour test.
//
// One workgroup per spectrum; thread l owns pixels [17 l, 17 l + 17) (the
// layout of the fused pass), so a new mask can be written straight into its
// (o/w, W w^2) array.
#include "lasp_internal.h"

#include <type_traits>

namespace lasp {
namespace {

constexpr int kMaxDPasses = 20;

// The rows come and the mask goes through LDS in pixel order, so that every
// access to memory is coalesced (a lane's own 17 pixels would put the 64
// lanes of each access on 64 cache lines), and a pixel keeps two values in
// registers: its residual and the excess |eps| - f G that all tests use.
// Bound half by the rows' latency and half by VALU issue (FP64 tests), so the
// three rows' loads fly together, each |m_j - m_{j+1}| is formed once and the
// sum over all valid pixels takes no tests.  Measured at 16,384 x 3,900 (0.83
// GB), a call: 0.217 ms (3.8 TB/s), 0.232 with the rows one after another and
// each difference twice, 0.546 with lane-strided accesses and three values per
// pixel.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(4))) void k_clean(
    Geometry g, CleanArgs a) {
  constexpr int NW = BLOCK / 64;
  constexpr int kRow = kNPL * BLOCK;
  constexpr int kScr = NW * 512 * 2;  // floats of block_sum_lds' scratch
  __shared__ __align__(16) float sRow[kRow > kScr ? kRow : kScr];
  __shared__ double sRed[NW * 64];
  __shared__ double sOut[2];
  __shared__ int sCnt[2][NW];
  __shared__ uint32_t sFl[2][BLOCK];  // each thread's flags, two sets used in turn
  double *sScr = reinterpret_cast<double *>(sRow);
  const int spec = blockIdx.x;
  if (a.s.target && a.s.t[spec] >= a.s.target[spec]) return;  // a stopped fit keeps its mask
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int P = g.P;
  const int j0 = tid * kNPL;
  const size_t row = (size_t)spec * P;

  // the rows' loads fly together, then each row goes through LDS: the lane's
  // pixels and the two beside them
  float xm[kNPL], xo[kNPL], xi[kNPL];
#pragma unroll
  for (int i = 0; i < kNPL; ++i) xm[i] = a.model[row + min(tid + i * BLOCK, P - 1)];
#pragma unroll
  for (int i = 0; i < kNPL; ++i) xo[i] = a.obs[row + min(tid + i * BLOCK, P - 1)];
#pragma unroll
  for (int i = 0; i < kNPL; ++i) xi[i] = a.ivar[row + min(tid + i * BLOCK, P - 1)];
  auto turn = [&](const float (&x)[kNPL], float (&v)[kNPL + 2]) {
#pragma unroll
    for (int i = 0; i < kNPL; ++i) sRow[tid + i * BLOCK] = x[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kNPL; ++i) v[i + 1] = sRow[j0 + i];
    v[0] = sRow[max(j0 - 1, 0)];
    v[kNPL + 1] = sRow[min(j0 + kNPL, kRow - 1)];
    __syncthreads();  // read before the next row comes
  };
  float m[kNPL + 2], o[kNPL + 2], iv[kNPL + 2];
  turn(xm, m);
  turn(xo, o);
  turn(xi, iv);
  double eps[kNPL], exc[kNPL];  // residual (0 where invalid), |residual| - f G
  double el = 0.0, er = 0.0;    // residuals of pixels j0 - 1 and j0 + 17
  uint32_t valid = 0;
  const double f = (double)a.f_shift;
  double gl = j0 > 0 ? fabs((double)m[1] - (double)m[0]) : 0.0;
#pragma unroll
  for (int i = -1; i <= kNPL; ++i) {
    const int j = j0 + i;
    const float ov = o[i + 1], wv = iv[i + 1];
    const bool ok = j >= 0 && j < P && isfinite(ov) && isfinite(wv) && wv > 0.f;
    const double e = ok ? (double)ov - (double)m[i + 1] : 0.0;
    if (i < 0) {
      el = e;
    } else if (i == kNPL) {
      er = e;
    } else {
      if (ok) valid |= 1u << i;
      eps[i] = e;
      // flux gradient G_j = max(|m_j - m_{j-1}|, |m_j - m_{j+1}|), ends use one side
      const double gr = j + 1 < P ? fabs((double)m[i + 1] - (double)m[i + 2]) : 0.0;
      exc[i] = fma(-f, fmax(gl, gr), fabs(e));
      gl = gr;
    }
  }

  int slot = 0;
  auto count = [&](uint32_t flags) {  // flagged pixels of the spectrum
    slot ^= 1;
    const int c = wave_sum((int)__popc(flags));
    if (lane == 0) sCnt[slot][wave] = c;
    __syncthreads();
    int t = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += sCnt[slot][w];
    return t;
  };
  // sample standard deviation of eps over the selected pixels (all: the valid
  // ones; the others' residuals are zero)
  auto stats = [&](auto all, uint32_t sel, int n) {
    double acc[1] = {0.0};
#pragma unroll
    for (int i = 0; i < kNPL; ++i)
      if (all.value || (sel >> i & 1u)) acc[0] += eps[i];
    block_sum_lds<NW, 1>(acc, sScr, sRed, sOut, lane, wave);
    const double mean = n > 0 ? sOut[0] / (double)n : 0.0;
    double v[1] = {0.0};
#pragma unroll
    for (int i = 0; i < kNPL; ++i)
      if (sel >> i & 1u) v[0] += (eps[i] - mean) * (eps[i] - mean);
    block_sum_lds<NW, 1>(v, sScr, sRed, sOut + 1, lane, wave);
    return n > 1 ? sqrt(sOut[1] / ((double)n - 1.0)) : 0.0;
  };
  const int nv = count(valid);  // its barrier also ends the last row's reads
  const double sigma = stats(std::true_type{}, valid, nv);

  // B with the relaxed thresholds k = 3, 4, 5, 7 (the last one stands if
  // every count is above 3 %)
  uint32_t bout = 0;
  for (int q = 0; q < 4; ++q) {
    const double k = q == 0 ? 3.0 : (q == 1 ? 4.0 : (q == 2 ? 5.0 : 7.0));
    bout = 0;
#pragma unroll
    for (int i = 0; i < kNPL; ++i)
      if ((valid >> i & 1u) && exc[i] > k * sigma) bout |= 1u << i;
    if ((double)count(bout) <= 0.03 * (double)nv) break;
  }

  // flags of the pixels beside the lane's, from the neighbouring threads
  int set = 0;
  auto beside = [&](uint32_t flags, uint32_t &left, uint32_t &right) {
    set ^= 1;
    sFl[set][tid] = flags;
    __syncthreads();
    left = tid > 0 ? sFl[set][tid - 1] >> (kNPL - 1) & 1u : 0u;
    right = tid + 1 < BLOCK ? sFl[set][tid + 1] & 1u : 0u;
  };
  uint32_t bl, br;
  beside(bout, bl, br);
  // C: neighbours of B outliers above 2 sigma
  uint32_t cout = 0;
  {
    const uint32_t near = (bout << 1 | bl) | (bout >> 1 | br << (kNPL - 1));
#pragma unroll
    for (int i = 0; i < kNPL; ++i)
      if ((valid & near) >> i & 1u && exc[i] > 2.0 * sigma) cout |= 1u << i;
  }
  const uint32_t kept = valid & ~bout & ~cout;
  const double sigma2 = stats(std::false_type{}, kept, count(kept));

  // D: grow from the outliers through same-sign, not larger neighbours; the
  // pixels that may join, by which side
  uint32_t from_l = 0, from_r = 0;
#pragma unroll
  for (int i = 0; i < kNPL; ++i) {
    const double es = i > 0 ? eps[i > 0 ? i - 1 : 0] : el;
    const double et = i < kNPL - 1 ? eps[i < kNPL - 1 ? i + 1 : i] : er;
    const bool may = (valid >> i & 1u) && exc[i] > sigma2;
    if (may && es * eps[i] > 0.0 && fabs(eps[i]) <= fabs(es)) from_l |= 1u << i;
    if (may && et * eps[i] > 0.0 && fabs(eps[i]) <= fabs(et)) from_r |= 1u << i;
  }
  uint32_t dout = 0;
  for (int pass = 0; pass < kMaxDPasses; ++pass) {
    const uint32_t out = (bout | cout | dout) & valid;
    uint32_t ol, orr;
    beside(out, ol, orr);
    const uint32_t nd =
        dout | (from_l & (out << 1 | ol)) | (from_r & (out >> 1 | orr << (kNPL - 1)));
    const int changed = __syncthreads_or(nd != dout);
    dout = nd;
    if (!changed) break;
  }

  // outputs: keep flags, the new weights of the fused pass, n_eff
  const uint32_t masked = (bout | cout | dout) & valid;
  const int n_kept = count(valid & ~masked);
  if (a.keep_out) {
    uint8_t *sKeep = reinterpret_cast<uint8_t *>(sRow);  // free: the sums above are done
#pragma unroll
    for (int i = 0; i < kNPL; ++i) sKeep[j0 + i] = (masked >> i & 1u) ? 0 : 1;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kNPL; ++i) {
      const int j = tid + i * BLOCK;
      if (j < P) a.keep_out[row + j] = sKeep[j];
    }
  }
  if (a.s.ow) {
    const float w = a.s.wscale[spec];
    const float w2 = w * w;
    float2 *dst = a.s.ow + (size_t)spec * kNPL * BLOCK + tid;
#pragma unroll
    for (int i = 0; i < kNPL; ++i)
      if (valid >> i & 1u) dst[i * BLOCK].y = (masked >> i & 1u) ? 0.f : iv[i + 1] * w2;
    if (tid == 0) a.s.neff[spec] = n_kept;
  }
  if (a.masked_out && tid == 0) a.masked_out[spec] = nv - n_kept;
}

}  // namespace

hipError_t launch_clean(const Geometry &g, const CleanArgs &a, hipStream_t st) {
  switch (g.block) {
    case 128: hipLaunchKernelGGL(k_clean<128>, dim3(g.B), dim3(128), 0, st, g, a); break;
    case 256: hipLaunchKernelGGL(k_clean<256>, dim3(g.B), dim3(256), 0, st, g, a); break;
    case 512: hipLaunchKernelGGL(k_clean<512>, dim3(g.B), dim3(512), 0, st, g, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace lasp
