// Once-per-fit preparation of each spectrum: pixel weights, the flux weight
// w of Eq. 6, the lane-major (o/w, W w^2) layout read by the fused pass, and
// the initial Adam state.
#include "lasp_internal.h"

namespace lasp {
namespace {

// Bound by memory: each row is read once into registers (17 pixels per
// thread, all loads in flight) and the layout is written once, through LDS.
// Measured at 65,536 x 3,900 (2.04 GB in, 2.28 GB out): 0.803 ms (5.4 TB/s),
// against 1.841 ms when four radix-select passes over LDS keys found the
// weight and the rows were read a second time for the layout.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_prepare(Geometry g, State s, const float *obs,
                                                   const float *ivar, const float *init,
                                                   double blo0, double blo1, double blo2,
                                                   double blo3, double blo4, double bhi0,
                                                   double bhi1, double bhi2, double bhi3,
                                                   double bhi4, float quantile, int init_state,
                                                   int target_steps) {
  __shared__ __align__(16) float2 stage[kNPL * BLOCK];
  __shared__ uint32_t scratch[kPrepScratch];
  const int spec = blockIdx.x;
  const int tid = threadIdx.x;
  const size_t row = (size_t)spec * g.P;
  float o[kNPL], iv[kNPL];
  const RowInfo r = prepare_row<BLOCK>(obs + row, ivar + row, g.P, quantile, scratch, o, iv);
  const float inv_w = 1.f / r.w;
  const float w2 = r.w * r.w;
#pragma unroll
  for (int i = 0; i < kNPL; ++i) stage[tid + i * BLOCK] = make_float2(o[i] * inv_w, iv[i] * w2);
  __syncthreads();
  // Lane-major layout for the fused pass: slot (i, lane) holds pixel
  // lane * kNPL + i, so a lane reads its pixels with coalesced loads.
  float2 *dst = s.ow + (size_t)spec * kNPL * BLOCK + tid;
#pragma unroll
  for (int i = 0; i < kNPL; ++i) dst[i * BLOCK] = stage[tid * kNPL + i];

  if (tid == 0) {
    uint32_t st = 0;
    if (r.any_bad) st |= kStNonfinite;
    if (r.n_eff <= kNP + g.nd) st |= kStNoData;
    s.status[spec] = st;
    s.neff[spec] = r.n_eff;
    s.wscale[spec] = r.w;
    if (init_state) {
      const double lo[5] = {blo0, blo1, blo2, blo3, blo4};
      const double hi[5] = {bhi0, bhi1, bhi2, bhi3, bhi4};
      for (int t = 0; t < kNP; ++t) {
        double th = (double)init[(size_t)spec * kNP + t];
        if (t == 0) th = log10(th);
        s.u[(size_t)spec * kNP + t] = (float)(2.0 * (th - lo[t]) / (hi[t] - lo[t]) - 1.0);
        s.m[(size_t)spec * kNP + t] = 0.f;
        s.v[(size_t)spec * kNP + t] = 0.f;
      }
      s.t[spec] = 0;
      if (s.target) s.target[spec] = target_steps;
      if (s.nrise) s.nrise[spec] = 0;
    }
  }
}

// Physical parameters, status and chi2 at the end of a fit.  OUT_OF_BOX is
// replaced by that of the returned parameters.
__global__ void k_finalize(Geometry g, State s, double blo0, double blo1, double blo2, double blo3,
                           double blo4, double bhi0, double bhi1, double bhi2, double bhi3,
                           double bhi4, float *out_params, uint32_t *status_out,
                           double *chi2_out, int32_t *steps_out) {
  const int spec = blockIdx.x * blockDim.x + threadIdx.x;
  if (spec >= g.B) return;
  const double lo[5] = {blo0, blo1, blo2, blo3, blo4};
  const double hi[5] = {bhi0, bhi1, bhi2, bhi3, bhi4};
  uint32_t st = (s.status[spec] & ~kStOutOfBox) | box_bit(s.u + (size_t)spec * kNP);
  for (int t = 0; t < kNP; ++t) {
    const double u = (double)s.u[(size_t)spec * kNP + t];
    double th = lo[t] + 0.5 * (u + 1.0) * (hi[t] - lo[t]);
    if (t == 0) th = exp10(th);
    out_params[(size_t)spec * kNP + t] = (float)th;
  }
  s.status[spec] = st;
  if (status_out) status_out[spec] = st;
  if (chi2_out) chi2_out[spec] = s.chi2[spec];
  if (steps_out) steps_out[spec] = s.t[spec];
}

// The spectra still taking steps, in index order within each Teff regime
// (with several emulator classes: cool, cool/warm blend, warm, warm/hot
// blend, hot, from the current parameters), regimes in that order, so that
// the contraction tiles mostly hold one regime.  Each thread counts the
// active spectra of its contiguous chunk per regime, workgroup-wide scans of
// the counts give each chunk's first position in each regime, and each
// thread writes its chunk.  One workgroup of 1024 threads.
__global__ __launch_bounds__(1024) void k_compact(Geometry g, State s, int *order,
                                                  int *n_active) {
  constexpr int kKeys = 5;
  __shared__ int cnt[kKeys][1024];
  __shared__ int first[kKeys + 1];
  const int t = threadIdx.x;
  const int nk = g.n_classes > 1 ? kKeys : 1;
  // regime boundaries in the normalised log Teff coordinate
  double ue[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) ue[e] = (log10(g.edges[e]) - g.lt_lo) / g.lt_half - 1.0;
  auto key = [&](int i) {
    if (nk == 1) return 0;
    const double u1 = s.u[(size_t)i * kNP];
    int k = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) k += u1 > ue[e] ? 1 : 0;
    return k;
  };
  const int chunk = (g.B + 1023) / 1024;
  const int b0 = min(t * chunk, g.B), b1 = min(b0 + chunk, g.B);
  int c[kKeys] = {0, 0, 0, 0, 0};
  for (int i = b0; i < b1; ++i) {
    if (!slot_active(s, i)) continue;
    const int k = key(i);
#pragma unroll
    for (int q = 0; q < kKeys; ++q) c[q] += q == k ? 1 : 0;
  }
#pragma unroll
  for (int q = 0; q < kKeys; ++q) cnt[q][t] = c[q];
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {  // inclusive scans
    int v[kKeys];
#pragma unroll
    for (int q = 0; q < kKeys; ++q) v[q] = (t >= off && q < nk) ? cnt[q][t - off] : 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kKeys; ++q) cnt[q][t] += v[q];
    __syncthreads();
  }
  if (t == 0) {
    first[0] = 0;
    for (int q = 0; q < kKeys; ++q) first[q + 1] = first[q] + cnt[q][1023];
  }
  __syncthreads();
  int pos[kKeys];
#pragma unroll
  for (int q = 0; q < kKeys; ++q) pos[q] = first[q] + cnt[q][t] - c[q];
  for (int i = b0; i < b1; ++i) {
    if (!slot_active(s, i)) continue;
    const int k = key(i);
#pragma unroll
    for (int q = 0; q < kKeys; ++q)
      if (q == k) order[pos[q]++] = i;
  }
  if (t == 1023) *n_active = first[kKeys];
}

// Steps taken and stopped flag of each slot.
__global__ void k_progress(Geometry g, State s, int32_t *steps, int32_t *done) {
  const int spec = blockIdx.x * blockDim.x + threadIdx.x;
  if (spec >= g.B) return;
  const int t = s.t[spec];
  if (steps) steps[spec] = t;
  if (done) done[spec] = (s.target && t >= s.target[spec]) ? 1 : 0;
}

// Per-spectrum results of a forward evaluation whose outputs lie in the memory
// of its inputs or of one another: chi2, the objective J = chi2 / n_eff of
// Eq. 9 (read per spectrum), n_eff and status (with OUT_OF_BOX of the
// evaluated u), out of the scratch after the last kernel.
__global__ void k_outputs(Geometry g, State s, double *chi2_out, float *J_out, int32_t *neff_out,
                          uint32_t *status_out) {
  const int spec = blockIdx.x * blockDim.x + threadIdx.x;
  if (spec >= g.B) return;
  const double c = s.chi2[spec];
  const int n = s.neff[spec];
  const uint32_t st = (s.status[spec] & ~kStOutOfBox) | box_bit(s.u + (size_t)spec * kNP);
  if (chi2_out) chi2_out[spec] = c;
  if (J_out) J_out[spec] = n > 0 ? (float)(c / (double)n) : 0.f;
  if (neff_out) neff_out[spec] = n;
  if (status_out) status_out[spec] = st;
}

}  // namespace

hipError_t launch_prepare(const Geometry &g, const State &s, const float *obs, const float *ivar,
                          const float *init_params, const double *lo, const double *hi,
                          float weight_quantile, int init_state, int target_steps,
                          hipStream_t st) {
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(g.B), dim3(g.block), 0, st, g, s, obs, ivar, init_params,
                       lo[0], lo[1], lo[2], lo[3], lo[4], hi[0], hi[1], hi[2], hi[3], hi[4],
                       weight_quantile, init_state, target_steps);
    return hipGetLastError();
  };
  switch (g.block) {
    case 128: return go(k_prepare<128>);
    case 256: return go(k_prepare<256>);
    case 512: return go(k_prepare<512>);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_finalize(const Geometry &g, const State &s, const double *lo, const double *hi,
                           float *out_params, uint32_t *status_out, double *chi2_out,
                           int32_t *steps_out, hipStream_t st) {
  const int bs = 256;
  hipLaunchKernelGGL(k_finalize, dim3((g.B + bs - 1) / bs), dim3(bs), 0, st, g, s, lo[0], lo[1],
                     lo[2], lo[3], lo[4], hi[0], hi[1], hi[2], hi[3], hi[4], out_params,
                     status_out, chi2_out, steps_out);
  return hipGetLastError();
}

hipError_t launch_compact(const Geometry &g, const State &s, int *order, int *n_active,
                          hipStream_t st) {
  hipLaunchKernelGGL(k_compact, dim3(1), dim3(1024), 0, st, g, s, order, n_active);
  return hipGetLastError();
}

hipError_t launch_progress(const Geometry &g, const State &s, int32_t *steps, int32_t *done,
                           hipStream_t st) {
  const int bs = 256;
  hipLaunchKernelGGL(k_progress, dim3((g.B + bs - 1) / bs), dim3(bs), 0, st, g, s, steps, done);
  return hipGetLastError();
}

hipError_t launch_outputs(const Geometry &g, const State &s, double *chi2_out, float *J_out,
                          int32_t *neff_out, uint32_t *status_out, hipStream_t st) {
  const int bs = 256;
  hipLaunchKernelGGL(k_outputs, dim3((g.B + bs - 1) / bs), dim3(bs), 0, st, g, s, chi2_out, J_out,
                     neff_out, status_out);
  return hipGetLastError();
}

}  // namespace lasp
