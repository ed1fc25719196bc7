// Preparation of one spectrum by one workgroup, shared by k_prepare and the
// one-shot passes: pixel weights, n_eff and the flux weight w of Eq. 6 (a
// flux quantile, Section 3.3 "Setting spectral weighting factors").
#pragma once

#include "lasp_internal.h"

namespace lasp {

__device__ inline bool pixel_ok(float o, float iv) {
  return isfinite(o) && isfinite(iv) && iv > 0.f;
}

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

// Scratch of the preparation in LDS: 256 counters, then the reductions.
constexpr int kPrepScratch = 256 + 2 + 8 + 3 * 8;  // 32-bit words

// k-th smallest (0-based) flux among the valid pixels of one spectrum, by a
// four-pass 8-bit radix select over the order-preserving keys (in LDS,
// kNoKey for invalid pixels).  Each pass counts the candidates' digits into
// 256 bins (a wave whose candidates all share one digit adds them with one
// atomic), then every thread takes its bins in a block-wide prefix sum and
// the one thread whose bin holds the k-th candidate records the digit and
// the rank within it.
template <int BLOCK>
__device__ float block_select(const uint32_t *keys, int P, uint32_t k, uint32_t *hist,
                              uint32_t *sh) {
  constexpr int kOwn = BLOCK >= 256 ? 1 : 256 / BLOCK;  // bins per thread (threads past 256: none)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t *wsum = sh + 2;  // [BLOCK / 64] totals of each wave's bins
  uint32_t prefix = 0, mask = 0;
  for (int shift = 24; shift >= 0; shift -= 8) {
    for (int b = tid; b < 256; b += BLOCK) hist[b] = 0;
    __syncthreads();
    for (int j = tid; j < P; j += BLOCK) {
      const uint32_t key = keys[j];
      const bool take = key != kNoKey && (key & mask) == prefix;
      const uint32_t bin = (key >> shift) & 255u;
      const uint64_t tk = __ballot(take);
      if (tk == 0) continue;
      const int first = __ffsll((unsigned long long)tk) - 1;
      const uint32_t b0 = __shfl(bin, first);
      if (__ballot(take && bin == b0) == tk) {
        if (lane == first) atomicAdd(&hist[b0], (uint32_t)__popcll(tk));
      } else if (take) {
        atomicAdd(&hist[bin], 1u);
      }
    }
    __syncthreads();
    uint32_t h[kOwn], mine = 0;
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
      h[q] = tid * kOwn + q < 256 ? hist[tid * kOwn + q] : 0u;
      mine += h[q];
    }
    uint32_t incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o);
      if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += wsum[w];
    uint32_t below = incl - mine;
    // bins 0..254 hold the k-th candidate when below <= k < below + h; bin
    // 255 takes whatever rank is past bin 254
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
      const int bin = tid * kOwn + q;
      if (bin < 256 && below <= k && (bin == 255 || k < below + h[q])) {
        sh[0] = (uint32_t)bin;
        sh[1] = k - below;
      }
      below += h[q];
    }
    __syncthreads();
    prefix |= sh[0] << shift;
    mask |= 255u << shift;
    k = sh[1];
    __syncthreads();
  }
  return funkey(prefix);
}

// The (k+1)-th smallest valid flux right after block_select(k) returned key0
// (its last pass left the digit and the rank in sh[0], sh[1] and the count of
// that exact key in hist): key0 again if another pixel holds it, else the
// smallest valid key above key0.
template <int BLOCK>
__device__ float block_select_next(const uint32_t *keys, int P, uint32_t key0,
                                   const uint32_t *hist, uint32_t *sh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t *wmin = sh + 2;  // [BLOCK / 64]
  if (sh[1] + 1 < hist[sh[0]]) return funkey(key0);  // block uniform
  uint32_t m = kNoKey;  // above every valid key
  for (int j = tid; j < P; j += BLOCK) {
    const uint32_t key = keys[j];
    if (key > key0) m = min(m, key);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = min(m, (uint32_t)__shfl_xor(m, o));
  __syncthreads();  // every thread has read sh and hist
  if (lane == 0) wmin[wave] = m;
  __syncthreads();
  m = wmin[0];
#pragma unroll
  for (int w = 1; w < BLOCK / 64; ++w) m = min(m, wmin[w]);
  __syncthreads();
  return funkey(m);
}

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
// counts over registers (two compares and two scalar population counts per
// pixel) on a spectrum.  Where the bracket does not close -- order
// statistics on both sides of an end or within 2^-12 of it, nonpositive or
// widely scattered fluxes -- q is formed from the order statistics of a
// radix select over keys in LDS (`keys`, P words).
//
// Every thread of the workgroup gets the same RowInfo.  scratch: kPrepScratch
// words of LDS; keys and scratch are free again after a barrier.
template <int BLOCK>
__device__ inline RowInfo prepare_row(const float *o_row, const float *i_row, int P, float quantile,
                                      uint32_t *keys, uint32_t *scratch, float (&o)[kNPL],
                                      float (&iv)[kNPL]) {
  constexpr int NW = BLOCK / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t *hist = scratch, *sh = scratch + 256;
  int *red_n = reinterpret_cast<int *>(scratch + 256 + 2 + 8);  // [3][8]
  int *red_b = red_n + 8;
  float *red_s = reinterpret_cast<float *>(red_n + 16);
#pragma unroll
  for (int i = 0; i < kNPL; ++i) {
    const int j = tid + i * BLOCK;
    o[i] = j < P ? o_row[j] : 0.f;
    iv[i] = j < P ? i_row[j] : 0.f;
  }
  int n = 0;
  uint64_t bad = 0;
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < kNPL; ++i) {
    bad |= __ballot(!isfinite(o[i]) || !isfinite(iv[i]));
    const bool ok = pixel_ok(o[i], iv[i]);
    n += __popcll(__ballot(ok));
    o[i] = ok ? o[i] : 0.f;
    iv[i] = ok ? iv[i] : 0.f;
    sum += o[i];
  }
  sum = wave_sum(sum);
  if (lane == 0) {
    red_n[wave] = n;
    red_b[wave] = bad != 0 ? 1 : 0;
    red_s[wave] = sum;
  }
  __syncthreads();
  RowInfo r{0, 0, 1.f};
  sum = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    r.n_eff += red_n[w];
    r.any_bad |= (uint32_t)red_b[w];
    sum += red_s[w];
  }
  r.n_eff = __builtin_amdgcn_readfirstlane(r.n_eff);
  if (!(quantile > 0.f) || r.n_eff == 0) return r;

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
        const float x = iv[i] > 0.f ? o[i] : INFINITY;
        c_lo += __popcll(__ballot(x < lo));
        c_hi += __popcll(__ballot(x <= hi));
      }
      __syncthreads();  // the previous counts have been read
      if (lane == 0) {
        red_n[wave] = c_lo;
        red_b[wave] = c_hi;
      }
      __syncthreads();
      c_lo = c_hi = 0;
#pragma unroll
      for (int q = 0; q < NW; ++q) {
        c_lo += red_n[q];
        c_hi += red_b[q];
      }
      c_lo = __builtin_amdgcn_readfirstlane(c_lo);
      c_hi = __builtin_amdgcn_readfirstlane(c_hi);
      if ((uint32_t)c_lo <= k0 && k1 < (uint32_t)c_hi) {
        w = exp2f((float)b);
        found = true;
        break;
      }
      const int step = k0 < (uint32_t)c_lo ? -1 : 1;
      go = dir == 0 || step == dir;  // past the quantile: the ends part it
      dir = step;
      b += step;
    }
  }
  if (!found) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kNPL; ++i) {
      const int j = tid + i * BLOCK;
      if (j < P) keys[j] = iv[i] > 0.f ? fkey(o[i]) : kNoKey;
    }
    __syncthreads();
    const float v0 = block_select<BLOCK>(keys, P, k0, hist, sh);
    float q = v0;
    if (k1 > k0) {
      const float v1 = block_select_next<BLOCK>(keys, P, fkey(v0), hist, sh);
      q = v0 + frac * (v1 - v0);
    }
    if (q > 0.f && isfinite(q)) w = exp2f(rintf(log2f(q)));
  }
  if (!(w > 0.f) || !isfinite(w) || !isfinite(1.f / (w * w))) w = 1.f;
  r.w = w;
  return r;
}

}  // namespace lasp
