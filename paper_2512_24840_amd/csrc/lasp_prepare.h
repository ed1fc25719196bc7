// Preparation of one spectrum by one workgroup, shared by k_prepare and the
// one-shot passes: pixel weights, n_eff and the flux weight w of Eq. 6 (a
// flux quantile, Section 3.3 "Setting spectral weighting factors").
#pragma once

#include "lasp_internal.h"

namespace lasp {

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
// counts over registers (four operations per pixel) on a spectrum.  Where
// the bracket does not close -- order statistics on both sides of an end or
// within 2^-12 of it, nonpositive or widely scattered fluxes -- q is formed
// from the order statistics themselves, found bit by bit by the same kind of
// counts over order-preserving keys.
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
#pragma unroll
  for (int i = 0; i < kNPL; ++i) {
    const int j = min(tid + i * BLOCK, P - 1);
    o[i] = o_row[j];
    iv[i] = i_row[j];
  }
  int n = 0;
  float sum = 0.f, fin = 0.f;  // fin: NaN once a value is not finite
#pragma unroll
  for (int i = 0; i < kNPL; ++i) {
    fin = fmaf(o[i], 0.f, fmaf(iv[i], 0.f, fin));
    const bool ok = isfinite(o[i]) && isfinite(iv[i]) && iv[i] > 0.f && tid + i * BLOCK < P;
    n += ok ? 1 : 0;
    sum += ok ? o[i] : 0.f;
    o[i] = ok ? o[i] : INFINITY;  // above every valid flux in the counts
    iv[i] = ok ? iv[i] : 0.f;
  }
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
#pragma unroll
      for (int i = 0; i < kNPL; ++i) {
        c_lo += o[i] < lo ? 1 : 0;
        c_hi += o[i] <= hi ? 1 : 0;
      }
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
#pragma unroll
      for (int i = 0; i < kNPL; ++i) c += __float_as_uint(o[i]) < t ? 1 : 0;
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

}  // namespace lasp
