// Interpolator contractions on the matrix cores (Eq. 1 read as a matrix
// product, F' = Phi(u) B, with B the [20 x (P+2M)] coefficient spectra) and
// the adjoint contraction Phi-bar = F-bar' B^T fused with the Adam update of
// Section 2.2 stage 8.
//
// v_mfma_f32_16x16x4f32 operand layout (wave64, one block):
//   A[i][k]: lane i + 16 k      B[k][j]: lane j + 16 k
//   D[i][j]: lane j + 16 (i / 4), register i % 4
// v_mfma_f32_16x16x32_bf16: lane l supplies row i = l % 16 of A (column
// j = l % 16 of B) with eight k values; A and B use the same k assignment,
// so the sum over k does not depend on which eight each lane carries.
//
// BF16x3: x = x_hi + x_lo with x_hi = bf16(x), x_lo = bf16(x - x_hi); a
// product is a_hi b_hi + a_hi b_lo + a_lo b_hi (the dropped a_lo b_lo is
// 2^-16 relative), accumulated in FP32.  In the forward contraction the
// constant monomial's row (phi_0 = 1) is added in FP32 exactly and only
// rows 1..19 go through BF16x3.
#include <algorithm>

#include "lasp_internal.h"

namespace lasp {
namespace {

constexpr int kFwdTiles = 8;  // 16-pixel tiles per wave in the forward GEMM
template <int V>
struct IntC {
  static constexpr int value = V;
};

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short ushort8 __attribute__((ext_vector_type(8)));

// x = hi + lo in bf16, rounded to nearest even (finite inputs).
__device__ inline void split8(const float *x, bf16x8 &hi, bf16x8 &lo) {
#pragma unroll
  for (int e = 0; e < 8; ++e) hi[e] = (__bf16)x[e];
  const ushort8 h = __builtin_bit_cast(ushort8, hi);
#pragma unroll
  for (int e = 0; e < 8; ++e) lo[e] = (__bf16)(x[e] - __uint_as_float((uint32_t)h[e] << 16));
}

// hi/lo copies of the padded basis in the products' operand order, 16 bytes a
// lane and a wave's load contiguous.  Adjoint contraction: of each 32 columns,
// rows 0-15 by lane (row + 16 kq: columns 8 kq .. + 7), then of all, rows 16-19
// by row - 16 + 4 kq.  Forward: of each 16 columns, lane (column + 16 kq) holds
// rows 8 kq .. + 7 (rows 1..19, zeros elsewhere).  Grid: (ldF / 256, 20 rows +
// 4 quarters): 5 us for 4,096 columns, 15 with one thread for all of a column.
__global__ __launch_bounds__(256) void k_split_basis(Geometry g, State s) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  float x[8];
  ushort8 *hi, *lo;
  if (blockIdx.y < kNB) {
    const int k = blockIdx.y;
    if (j >= g.ldF / 8) return;
    const float4 *p = reinterpret_cast<const float4 *>(s.basis + (size_t)k * g.ldF) + 2 * j;
    const float4 x0 = p[0], x1 = p[1];
    x[0] = x0.x; x[1] = x0.y; x[2] = x0.z; x[3] = x0.w;
    x[4] = x1.x; x[5] = x1.y; x[6] = x1.z; x[7] = x1.w;
    const int chunk = j >> 2, kq = j & 3;
    const size_t at = k < 16 ? (size_t)chunk * 64 + 16 * kq + k
                             : (size_t)2 * g.ldF + (size_t)chunk * 16 + 4 * kq + (k - 16);
    hi = reinterpret_cast<ushort8 *>(s.basis_hi) + at;
    lo = reinterpret_cast<ushort8 *>(s.basis_lo) + at;
  } else {
    const int kq = blockIdx.y - kNB;
    if (j >= g.ldF) return;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = 8 * kq + e;
      x[e] = k >= 1 && k < kNB ? s.basis[(size_t)k * g.ldF + j] : 0.f;
    }
    const size_t at = (size_t)(j >> 4) * 64 + 16 * kq + (j & 15);
    hi = reinterpret_cast<ushort8 *>(s.basis_thi) + at;
    lo = reinterpret_cast<ushort8 *>(s.basis_tlo) + at;
  }
  bf16x8 h, l;
  split8(x, h, l);
  *hi = __builtin_bit_cast(ushort8, h);
  *lo = __builtin_bit_cast(ushort8, l);
}

// Output staging of the forward contraction: a workgroup's 16 rows x 512
// columns pass through LDS so that each row leaves as contiguous 1 KB runs
// (the MFMA result layout alone gives 64-byte pieces of 16 rows).
constexpr int kFwdCols = 4 * 16 * kFwdTiles;  // columns per workgroup
constexpr int kFwdLd = kFwdCols + 4;           // LDS row stride (floats)

__device__ inline void fwd_stage(float *sT, int wave, int lane, int n, const floatx4 &v) {
  const int j = lane & 15, kq = lane >> 4;
  *reinterpret_cast<float4 *>(sT + j * kFwdLd + wave * 16 * kFwdTiles + 16 * n + 4 * kq) =
      make_float4(v[0], v[1], v[2], v[3]);
}

// F' rows of the block's 16 launch rows r0 + j: row r (entry r / rps of the
// work list, derivative row r % rps) lands in F' row spec * rps + r % rps.
// Threads 0..15 write dst; a barrier must follow before fwd_store.
__device__ inline void fwd_dst_rows(const State &s, int r0, int rows, int rps, int *dst) {
  const int j = threadIdx.x;
  if (j >= 16 || r0 + j >= rows) return;
  const int r = r0 + j;
  if (!s.order) {
    dst[j] = r;  // no work list: rows in place
  } else {
    const int e = r / rps;
    dst[j] = s.order[e] * rps + (r - e * rps);
  }
}

__device__ inline void fwd_store(const Geometry &g, const State &s, const float *sT,
                                 const int *dst, int r0, int rows) {
  const int c_base = blockIdx.x * kFwdCols;
#pragma unroll
  for (int q = 0; q < 16 * kFwdCols / 4 / 256; ++q) {
    const int e = threadIdx.x + 256 * q;
    const int r = e / (kFwdCols / 4), c4 = e - r * (kFwdCols / 4);
    const int col = c_base + 4 * c4;
    if (r0 + r < rows && col < g.ldF)
      *reinterpret_cast<float4 *>(s.fp + (size_t)dst[r] * g.ldF + col) =
          *reinterpret_cast<const float4 *>(sT + r * kFwdLd + 4 * c4);
  }
}

// Row tiles per workgroup of the forward GEMM, from the rows of the work list:
// enough that the workgroups are all resident at once (four per CU, by LDS),
// and the basis entries are read once for them.  3,900 px in FP32, one tile
// against this rule: 6,000 rows 27.2 and 25.0 us, 20,000 69.0 and 59.6, 65,536
// 275 and 192; with two tiles (4,096 rows) 21.0 both, so from three on.  The
// BF16x3 kernel (three workgroups per CU) takes 8 tiles at most: 65,536 rows
// 273 and 189 us, 208 with 16 tiles.  One tile over fixed slots of which some
// may be done (no work list), lest the active ones meet in few workgroups, and
// over three classes, whose basis entries do not fit the registers.
constexpr int kFwdResident = 1024;
constexpr int kFwdBf16Tiles = 8;
__host__ __device__ inline bool fwd_one_tile(const Geometry &g, const State &s) {
  return g.nb != kNB || (s.target && !s.order);
}
__device__ inline int fwd_row_tiles(const Geometry &g, const State &s, int rows, int most) {
  if (fwd_one_tile(g, s)) return 1;
  const int rounds = ((rows + 15) / 16 * (int)gridDim.x + kFwdResident - 1) / kFwdResident;
  return rounds < 3 ? 1 : min(rounds, most);
}

// BF16x3 variant of k_interp_fwd (same grid and output layout, the basis
// entries kept over the row tiles as there): 16,384 x 3,900 in 51 us (72).
// The constant row is one FP32 product on the matrix core, a fused
// multiply-add of the sum like any other step of its chain.
__global__ __launch_bounds__(256) void k_interp_fwd_bf16(Geometry g, State s, int rows_per_spec, int skip_done) {
  __shared__ __align__(16) float sT[16 * kFwdLd];
  __shared__ int dst[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rows = work_count(g, s) * rows_per_spec;
  const int row_tiles = fwd_row_tiles(g, s, rows, kFwdBf16Tiles);
  int r0 = blockIdx.y * 16 * row_tiles;
  if (r0 >= rows) return;  // past the work list (uniform over the block)
  const int r_end = min(rows, r0 + 16 * row_tiles);
  const int kq = lane >> 4;
  const int cbase = (blockIdx.x * 4 + wave) * (16 * kFwdTiles);
  bf16x8 a_hi[kFwdTiles], a_lo[kFwdTiles];
  float a0[kFwdTiles];  // row 0 of the basis, with the lanes of k = 0
#pragma unroll
  for (int n = 0; n < kFwdTiles; ++n) {
    const int c0 = min(cbase + 16 * n, g.ldF - 16);
    const size_t e = (size_t)c0 * 4 + lane;
    a_hi[n] = __builtin_bit_cast(bf16x8, reinterpret_cast<const ushort8 *>(s.basis_thi)[e]);
    a_lo[n] = __builtin_bit_cast(bf16x8, reinterpret_cast<const ushort8 *>(s.basis_tlo)[e]);
    a0[n] = kq == 0 ? s.basis[c0 + (lane & 15)] : 0.f;
  }
  for (; r0 < r_end; r0 += 16) {
    const int my_row = r0 + (lane & 15);
    if (skip_done && s.target) {
      bool any = false;
      for (int r = 0; r < 16; ++r) {
        const int row = r0 + r;
        any = any || (row < rows && slot_active(s, work_spec(s, row / rows_per_spec)));
      }
      if (!any) continue;  // (uniform over the block)
    }
    fwd_dst_rows(s, r0, rows, rows_per_spec, dst);
    bf16x8 b_hi, b_lo;
    float phi0 = 0.f;
    {
      float phi[32];
#pragma unroll
      for (int k = 0; k < 32; ++k) phi[k] = 0.f;
      if (my_row < rows) {
        const int e = my_row / rows_per_spec;
        const int t = my_row - e * rows_per_spec;
        feature_row(s.u + (size_t)work_spec(s, e) * kNP, t, phi);
      }
      phi0 = phi[0];
      phi[0] = 0.f;  // constant row added in FP32 below
      float sel[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float v = phi[e];
#pragma unroll
        for (int q = 1; q < 4; ++q)
          if (kq == q) v = phi[8 * q + e];
        sel[e] = v;
      }
      split8(sel, b_hi, b_lo);
    }
#pragma unroll
    for (int n = 0; n < kFwdTiles; ++n) {
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_lo[n], b_hi, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_hi[n], b_lo, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_hi[n], b_hi, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[n], phi0, acc, 0, 0, 0);
      fwd_stage(sT, wave, lane, n, acc);
    }
    __syncthreads();
    fwd_store(g, s, sT, dst, r0, rows);
    if (r0 + 16 < r_end) __syncthreads();  // the stage and dst are rewritten
  }
}

// F'[r][c] = sum_k Phi[r][k] basis[k][c] for r < rows (rows = B or 4B with
// derivative rows), k < NB (20, or 60 over three emulator classes).
// Grid: (ldF / (64 * kFwdTiles), workgroups for ceil(rows / 16) tiles).
//
// Bound by the stores of F'.  A tile needs 40 KB of basis entries and stores
// 32 KB, so (of one class) a workgroup keeps its basis entries in registers
// over several tiles: 65,536 x 3,900 in 192 us (5.6 TB/s) against 275 when
// each tile read them anew.
template <int NB>
__global__ __launch_bounds__(256) void k_interp_fwd(Geometry g, State s, int rows_per_spec, int skip_done) {
  __shared__ __align__(16) float sT[16 * kFwdLd];
  __shared__ int dst[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rows = work_count(g, s) * rows_per_spec;
  const int tiles = NB == kNB ? fwd_row_tiles(g, s, rows, 1 << 30) : 1;
  int r0 = blockIdx.y * 16 * tiles;
  if (r0 >= rows) return;  // past the work list (uniform over the block)
  const int r_end = NB == kNB ? min(rows, r0 + 16 * tiles) : r0 + 1;
  const int kq = lane >> 4;  // k offset inside a group of 4
  const int cbase = (blockIdx.x * 4 + wave) * (16 * kFwdTiles);
  float av[kFwdTiles][kNB / 4];  // NB == kNB: the wave's basis entries
  if constexpr (NB == kNB) {
#pragma unroll
    for (int n = 0; n < kFwdTiles; ++n)
#pragma unroll
      for (int kk = 0; kk < kNB / 4; ++kk)
        av[n][kk] = s.basis[(size_t)(4 * kk + kq) * g.ldF + min(cbase + 16 * n, g.ldF - 16) + (lane & 15)];
  }
  for (; r0 < r_end; r0 += 16) {
    const int my_row = r0 + (lane & 15);
    if (skip_done && s.target) {
      bool any = false;
      for (int r = 0; r < 16; ++r) {
        const int row = r0 + r;
        any = any || (row < rows && slot_active(s, work_spec(s, row / rows_per_spec)));
      }
      if (!any) continue;  // (uniform over the block)
    }
    fwd_dst_rows(s, r0, rows, rows_per_spec, dst);

    float bv[NB / 4];
    {
      float phi[NB];
#pragma unroll
      for (int k = 0; k < NB; ++k) phi[k] = 0.f;
      if (my_row < rows) {
        const int e = my_row / rows_per_spec;
        const int t = my_row - e * rows_per_spec;
        const float *ur = s.u + (size_t)work_spec(s, e) * kNP;
        if (NB == kNB)
          feature_row(ur, t, phi);
        else
          feature_row_classes(g, ur, t, phi);
      }
      // selects, not an indexed load: keeps phi in registers
#pragma unroll
      for (int kk = 0; kk < NB / 4; ++kk)
        bv[kk] = kq == 0 ? phi[4 * kk] : (kq == 1 ? phi[4 * kk + 1] : (kq == 2 ? phi[4 * kk + 2] : phi[4 * kk + 3]));
    }
    // products over feature groups KK0 .. KK0 + NKK - 1 (4 features each)
    auto run = [&](auto kk0, auto nkk) {
      constexpr int KK0 = decltype(kk0)::value, NKK = decltype(nkk)::value;
      for (int n = 0; n < kFwdTiles; ++n) {
        const int c0 = cbase + 16 * n;
        if (c0 >= g.ldF) break;
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = KK0; kk < KK0 + NKK; ++kk) {
          const float a = s.basis[(size_t)(4 * kk + kq) * g.ldF + c0 + (lane & 15)];
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, bv[kk], acc, 0, 0, 0);
        }
        fwd_stage(sT, wave, lane, n, acc);
      }
    };
    if constexpr (NB == kNB) {
#pragma unroll
      for (int n = 0; n < kFwdTiles; ++n) {
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < NB / 4; ++kk)
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[n][kk], bv[kk], acc, 0, 0, 0);
        fwd_stage(sT, wave, lane, n, acc);
      }
    } else {
      // an emulator class whose weight and weight derivative are zero in all
      // 16 rows of the tile (spectra of other Teff regimes) has an all-zero
      // feature block; its products would add exact zeros and are left out
      int mask = 0;
#pragma unroll
      for (int q = 0; q < kMaxClasses; ++q) {
        bool nz = false;
#pragma unroll
        for (int kk = 5 * q; kk < 5 * q + 5; ++kk) nz = nz || bv[kk] != 0.f;
        mask |= (__ballot(nz) != 0) << q;
      }
      switch (mask) {  // wave uniform; every wave of the block sees the same rows
        case 1: run(IntC<0>{}, IntC<5>{}); break;
        case 2: run(IntC<5>{}, IntC<5>{}); break;
        case 4: run(IntC<10>{}, IntC<5>{}); break;
        case 3: run(IntC<0>{}, IntC<10>{}); break;
        case 6: run(IntC<5>{}, IntC<10>{}); break;
        default: run(IntC<0>{}, IntC<15>{}); break;
      }
    }
    __syncthreads();
    fwd_store(g, s, sT, dst, r0, rows);
    if (r0 + 16 < r_end) __syncthreads();  // the stage and dst are rewritten
  }
}

// Gradient of J with respect to u from Phi-bar (pb, NB entries) and the
// fused pass's dJ/du4, dJ/du5, then the stopping rules and one Adam step of
// spectrum spec (or the gradient written out).
template <int NB>
__device__ inline void bwd_epilogue(const Geometry &g, const State &s, const AdamCfg &adam,
                                    int do_adam, float *grad_out, int spec, const float *pb) {
  float *u = s.u + (size_t)spec * kNP;
  float grad[kNP];
  float d[3][kNB];
  feature_derivs(u[0], u[1], u[2], d);
  if constexpr (NB == kNB) {
#pragma unroll
    for (int a = 0; a < 3; ++a) grad[a] = shape_gradient(pb, d[a]);
  } else {
    // d (sum_q w_q phi . Phi-bar_q) / d u_a: the class weights depend on u1
    float phi[kNB], w[kMaxClasses], dw[kMaxClasses];
    features(u[0], u[1], u[2], phi);
    class_weights(g, u[0], w, dw);
#pragma unroll
    for (int a = 0; a < 3; ++a) grad[a] = 0.f;
#pragma unroll
    for (int q = 0; q < kMaxClasses; ++q) {
      const float *pq = &pb[kNB * q];
      float sp = 0.f, sd0 = 0.f, sd1 = 0.f, sd2 = 0.f;
#pragma unroll
      for (int k = 0; k < kNB; ++k) {
        sp = fmaf(pq[k], phi[k], sp);
        sd0 = fmaf(pq[k], d[0][k], sd0);
        sd1 = fmaf(pq[k], d[1][k], sd1);
        sd2 = fmaf(pq[k], d[2][k], sd2);
      }
      grad[0] = fmaf(dw[q], sp, fmaf(w[q], sd0, grad[0]));
      grad[1] = fmaf(w[q], sd1, grad[1]);
      grad[2] = fmaf(w[q], sd2, grad[2]);
    }
  }
  grad[3] = s.g45[(size_t)spec * 2 + 0];
  grad[4] = s.g45[(size_t)spec * 2 + 1];
  if (grad_out) {
#pragma unroll
    for (int a = 0; a < kNP; ++a) grad_out[(size_t)spec * kNP + a] = grad[a];
  }
  bool take = do_adam && slot_active(s, spec);
  if (take && adam.stop_window > 0) {
    // stopping rules of stage 8 on ell_t = sqrt(chi2 / n_eff) after t steps:
    // a change below stop_tol over the last W steps, or a rise at each of
    // them (the ring holds ell of the last W step counts)
    const int t0 = s.t[spec], W = adam.stop_window;
    const int n = s.neff[spec];
    const double ell = n > 0 ? sqrt(s.chi2[spec] / (double)n) : 0.0;
    double *h = s.lhist + (size_t)spec * W;
    int rise = s.nrise[spec];
    if (t0 >= 1) rise = ell > h[(t0 - 1) % W] ? rise + 1 : 0;
    uint32_t bit = 0;
    if (t0 >= W && fabs(h[t0 % W] - ell) < (double)adam.stop_tol)
      bit = kStStopFlat;
    else if (rise >= W)
      bit = kStStopRising;
    s.nrise[spec] = rise;
    h[t0 % W] = ell;
    if (bit) {
      s.target[spec] = t0;
      s.status[spec] |= bit;
      take = false;
    }
  }
  if (take) {
    const int step = s.t[spec] + 1;
    s.t[spec] = step;
    if (adam.stop_window > 0 && step >= s.target[spec]) s.status[spec] |= kStNotConverged;
    float *m = s.m + (size_t)spec * kNP, *v = s.v + (size_t)spec * kNP;
    float ua[kNP], ma[kNP], va[kNP];  // all loads before the first store
#pragma unroll
    for (int a = 0; a < kNP; ++a) {
      ua[a] = u[a];
      ma[a] = m[a];
      va[a] = v[a];
    }
    const AdamStep as = adam_step(adam, step);
#pragma unroll
    for (int a = 0; a < kNP; ++a) {
      adam_update(adam, as, grad[a], ma[a], va[a], ua[a]);
      u[a] = ua[a];
      m[a] = ma[a];
      v[a] = va[a];
    }
  }
}

// BF16x3 variant of the adjoint contraction (one emulator class): one
// workgroup = 16 spectra; its four waves split the columns and combine
// through LDS.  Bound by the loads of F-bar' and their latency (two 1 KB loads
// a wave in flight; three chunks ahead gained nothing): 16,384 x 3,900 in 74 us
// (3.6 TB/s), 91 when F-bar' and the basis rows were read with a row per lane.
__global__ __launch_bounds__(256) void k_interp_bwd_bf16(Geometry g, State s, AdamCfg adam,
                                                         int do_adam, float *grad_out) {
  constexpr int NB = kNB;
  constexpr int NG = 2;
  constexpr int kLd = 36;  // row stride of a wave's [16][32] stage
  __shared__ __align__(16) float stage[4][16 * kLd];
  __shared__ float red[4][16][16 * NG];
  __shared__ float pb[16][NB];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int s0 = blockIdx.x * 16;
  const int count = work_count(g, s);
  if (s0 >= count) return;  // past the work list (uniform over the block)
  const int i_row = lane & 15;   // spectrum within the tile (A rows) / basis row (B cols)
  const int kq = lane >> 4;
  if (s.target) {  // the whole tile finished: nothing to do (uniform over the block)
    bool any = false;
    for (int r = 0; r < 16; ++r) any = any || (s0 + r < count && slot_active(s, work_spec(s, s0 + r)));
    if (!any) return;
  }

  floatx4 acc[NG];
#pragma unroll
  for (int q = 0; q < NG; ++q) acc[q] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int per_wave = g.ldF / 4;  // ldF is a multiple of 128
  const int cb = wave * per_wave;
  const int ce = cb + per_wave;
  const ushort8 *h0 = reinterpret_cast<const ushort8 *>(s.basis_hi) + lane;
  const ushort8 *l0 = reinterpret_cast<const ushort8 *>(s.basis_lo) + lane;
  const bool b_ok = i_row < NB - 16;  // the lanes of basis rows 16-19
  const size_t at1 = (size_t)2 * g.ldF + 4 * kq + (b_ok ? i_row : 0);
  const ushort8 *h1 = reinterpret_cast<const ushort8 *>(s.basis_hi) + at1;
  const ushort8 *l1 = reinterpret_cast<const ushort8 *>(s.basis_lo) + at1;
  const bf16x8 zero = __builtin_bit_cast(bf16x8, ushort8{0, 0, 0, 0, 0, 0, 0, 0});
  // F-bar' passes through LDS: eight lanes read 128 bytes of a row (read with
  // a row per lane, a load touches 16 cache lines with each quarter of the
  // wave), the next 32 columns while these are at work.
  float *stg = stage[wave];
  const int sr = lane >> 3, sc = 4 * (lane & 7);
  const float *rp[2];
  bool rv[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    rv[j] = s0 + 8 * j + sr < count;
    rp[j] = s.fbar + (size_t)work_spec(s, rv[j] ? s0 + 8 * j + sr : s0) * g.ldF + sc;
  }
  float4 fv[2];
  auto fetch = [&](int c) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
      fv[j] = rv[j] ? *reinterpret_cast<const float4 *>(rp[j] + c) : make_float4(0.f, 0.f, 0.f, 0.f);
  };
  fetch(cb);
  for (int c = cb; c < ce; c += 32) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
      *reinterpret_cast<float4 *>(stg + (8 * j + sr) * kLd + sc) = fv[j];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (c + 32 < ce) fetch(c + 32);
    const float4 x0 = *reinterpret_cast<const float4 *>(stg + i_row * kLd + 8 * kq);
    const float4 x1 = *reinterpret_cast<const float4 *>(stg + i_row * kLd + 8 * kq + 4);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const float fa[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
    bf16x8 a_hi, a_lo;
    split8(fa, a_hi, a_lo);
    const bf16x8 bh0 = __builtin_bit_cast(bf16x8, h0[2 * c]);
    const bf16x8 bl0 = __builtin_bit_cast(bf16x8, l0[2 * c]);
    bf16x8 bh1 = zero, bl1 = zero;
    if (b_ok) {
      bh1 = __builtin_bit_cast(bf16x8, h1[c / 2]);
      bl1 = __builtin_bit_cast(bf16x8, l1[c / 2]);
    }
    acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_lo, bh0, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_lo, bh1, acc[1], 0, 0, 0);
    acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_hi, bl0, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_hi, bl1, acc[1], 0, 0, 0);
    acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_hi, bh0, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_hi, bh1, acc[1], 0, 0, 0);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) red[wave][4 * kq + q][16 * gi + i_row] = acc[gi][q];
  __syncthreads();
  for (int e = threadIdx.x; e < 16 * NB; e += 256) {
    const int i = e / NB, k = e - i * NB;
    pb[i][k] = ((red[0][i][k] + red[1][i][k]) + red[2][i][k]) + red[3][i][k];
  }
  __syncthreads();

  const int t = threadIdx.x;
  if (t < 16 && s0 + t < count)
    bwd_epilogue<NB>(g, s, adam, do_adam, grad_out, work_spec(s, s0 + t), pb[t]);
}

// Phi-bar[s][k] = sum_c F-bar'[s][c] basis[k][c], then the gradient of
// J = chi2/n_eff with respect to u and one Adam step (or, with grad_out,
// the gradient written out and no update).  One workgroup = 32 spectra in
// two 16-row tiles; each of its eight waves covers ldF / 8 columns for both
// tiles, so one basis load feeds both, and the waves combine through LDS in
// a fixed order.  Basis rows go in groups of 16 (NG = 2 groups for 20 rows,
// 4 for 60); the loads of rows past NB are skipped and count as zero.
template <int NB>
__global__ __launch_bounds__(512) void k_interp_bwd(Geometry g, State s, AdamCfg adam,
                                                      int do_adam, float *grad_out) {
  constexpr int NG = (NB + 15) / 16;
  constexpr int NWV = 8;
  constexpr int kSLd = 36;                        // staging row stride (floats)
  constexpr int kStage = 36 * kSLd;               // one wave's [32 + 4 rows][32 columns]
  constexpr int kRed = 32 * 16 * NG;              // one wave's partial sums
  constexpr int kBuf = NWV * (kStage > kRed ? kStage : kRed);
  __shared__ __align__(16) float sbuf[kBuf];      // staging, then the partial sums
  __shared__ float pb[32][NB];
  auto red = reinterpret_cast<float (*)[32][16 * NG]>(sbuf);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int s0 = blockIdx.x * 32;
  const int count = work_count(g, s);
  if (s0 >= count) return;  // past the work list (uniform over the block)
  const int i_row = lane & 15;
  const int kq = lane >> 4;
  bool row_ok[2];
  const float *fb_row[2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    row_ok[rt] = s0 + 16 * rt + i_row < count;
    fb_row[rt] = s.fbar + (size_t)work_spec(s, row_ok[rt] ? s0 + 16 * rt + i_row : s0) * g.ldF;
  }
  bool b_ok[NG];
  const float *b_ptr[NG];
#pragma unroll
  for (int q = 0; q < NG; ++q) {
    b_ok[q] = 16 * q + i_row < NB;
    b_ptr[q] = s.basis + (size_t)(16 * q + (b_ok[q] ? i_row : 0)) * g.ldF;
  }
  if (s.target) {
    bool any = false;
    for (int r = 0; r < 32; ++r) any = any || (s0 + r < count && slot_active(s, work_spec(s, s0 + r)));
    if (!any) return;
  }
  floatx4 acc[2][NG];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int q = 0; q < NG; ++q) acc[rt][q] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int per_wave = g.ldF / NWV;  // ldF is a multiple of 128
  const int cb = wave * per_wave, ce = cb + per_wave;
  constexpr int kU = 2;  // 16-column MFMA blocks per stage
  // groups Q0 .. Q1 - 1 of 16 basis rows
  auto step = [&](auto q0, auto q1, const float4 (&fa)[2], const float4 (&bv)[NG]) {
    constexpr int Q0 = decltype(q0)::value, Q1 = decltype(q1)::value;
    float4 a[2];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) a[rt] = row_ok[rt] ? fa[rt] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int q = Q0; q < Q1; ++q) acc[rt][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[rt].x, bv[q].x, acc[rt][q], 0, 0, 0);
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int q = Q0; q < Q1; ++q) acc[rt][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[rt].y, bv[q].y, acc[rt][q], 0, 0, 0);
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int q = Q0; q < Q1; ++q) acc[rt][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[rt].z, bv[q].z, acc[rt][q], 0, 0, 0);
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int q = Q0; q < Q1; ++q) acc[rt][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[rt].w, bv[q].w, acc[rt][q], 0, 0, 0);
  };
  auto load = [&](auto q0, auto q1, int cc, float4 (&fa)[2], float4 (&bv)[NG]) {
    constexpr int Q0 = decltype(q0)::value, Q1 = decltype(q1)::value;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) fa[rt] = *reinterpret_cast<const float4 *>(fb_row[rt] + cc);
#pragma unroll
    for (int q = Q0; q < Q1; ++q) {
      if (16 * q + 16 <= NB || b_ok[q])
        bv[q] = *reinterpret_cast<const float4 *>(b_ptr[q] + cc);
      else
        bv[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  // F-bar' goes through this wave's LDS stage, 32 rows x 32 columns at a
  // time, read with row-contiguous loads (128-byte runs per row); the MFMA
  // operands (16 rows x 4 columns per lane group) come from LDS.  The next
  // stage's F-bar' and basis loads are in flight during this stage's
  // products.
  float *stg = sbuf + wave * kStage;
  const float *rp[4];
  bool rv[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int ri = 8 * j + (lane >> 3);
    rv[j] = s0 + ri < count;
    rp[j] = s.fbar + (size_t)work_spec(s, rv[j] ? s0 + ri : s0) * g.ldF + 4 * (lane & 7);
  }
  auto run = [&](auto q0, auto q1) {
    auto fetch = [&](int cc, float4 (&fv)[4], float4 (&bv)[kU][NG]) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        fv[j] = rv[j] ? *reinterpret_cast<const float4 *>(rp[j] + cc) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        float4 dummy[2];
        load(q0, q1, cc + 16 * u + 4 * kq, dummy, bv[u]);
      }
    };
    int c = cb;
    if (c + 16 * kU <= ce) {
      float4 fv[4], bv[kU][NG];
      fetch(c, fv, bv);
      for (; c + 16 * kU <= ce; c += 16 * kU) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          *reinterpret_cast<float4 *>(stg + (8 * j + (lane >> 3)) * kSLd + 4 * (lane & 7)) = fv[j];
        float4 bcur[kU][NG];
#pragma unroll
        for (int u = 0; u < kU; ++u)
#pragma unroll
          for (int q = 0; q < NG; ++q) bcur[u][q] = bv[u][q];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (c + 32 * kU <= ce) fetch(c + 16 * kU, fv, bv);  // next stage
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          float4 fa[2];
#pragma unroll
          for (int rt = 0; rt < 2; ++rt)
            fa[rt] = *reinterpret_cast<const float4 *>(stg + (16 * rt + i_row) * kSLd + 16 * u + 4 * kq);
          step(q0, q1, fa, bcur[u]);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
    for (; c < ce; c += 16) {
      float4 fa[2], bv[NG];
      load(q0, q1, c + 4 * kq, fa, bv);
      step(q0, q1, fa, bv);
    }
  };
  floatx4 acc4[4];   // NB == kNB: rows 16-19
  floatx16 acc16[2];  // NB == kNB: rows 0-15
  if constexpr (NB == kNB) {
    // Basis rows 0-15 as products of four 16x16x1 blocks, one per quarter of
    // the 16 columns: a lane's float4 is four steps of its block.  Rows 16-19
    // as sixteen 4x4x1 blocks, no zero rows: block b = g + 8 h (lanes 4b ..
    // 4b + 3) takes spectra 4g .. 4g + 3 and the h-th 16 columns of each
    // 32-column stage, so lane l supplies F-bar' of spectrum l & 31 and
    // basis row 16 + (l & 3), and accumulates spectra 4g + r x row 16 + (l & 3),
    // each float4 of the 16 columns in an accumulator of its own.
    //
    // So an entry of Phi-bar is, per wave, a few chains of fused multiply-adds
    // over the float4 at one place of every 16 (rows 0-15) or 32 (rows 16-19)
    // columns, added pairwise: the order in which a workgroup that holds one
    // spectrum can form it with coalesced loads (the fit kernel does, and its
    // fits are these bit for bit).  The products' rate is that of 16x16x4:
    // 65.3 us at 16,384 x 3,900 (64.8 in one chain), 211 at
    // 65,536 (200), 0.5 % of a pass.  One workgroup per CU
    // is no worse than two: held to 128 registers the kernel took 66 to 96 us
    // in several forms, and 73 with the basis rows staged through LDS.
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc16[rt][r] = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) acc4[q] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto step16 = [&](const float4 (&a)[2], const float4 &b) {
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) acc16[rt] = __builtin_amdgcn_mfma_f32_16x16x1f32(a[rt].x, b.x, acc16[rt], 0, 0, 0);
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) acc16[rt] = __builtin_amdgcn_mfma_f32_16x16x1f32(a[rt].y, b.y, acc16[rt], 0, 0, 0);
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) acc16[rt] = __builtin_amdgcn_mfma_f32_16x16x1f32(a[rt].z, b.z, acc16[rt], 0, 0, 0);
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) acc16[rt] = __builtin_amdgcn_mfma_f32_16x16x1f32(a[rt].w, b.w, acc16[rt], 0, 0, 0);
    };
    const int hh = lane >> 5, r4 = lane & 31, j4 = lane & 3;
    const float *b4 = s.basis + (size_t)(16 + j4) * g.ldF;
    const float *fb4row = s.fbar + (size_t)work_spec(s, s0 + r4 < count ? s0 + r4 : s0) * g.ldF;
    float *stg = sbuf + wave * kStage;
    uint32_t ro[4];  // row offsets in float4 (B ldF / 4, below 2^32)
    bool rv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int ri = 8 * j + (lane >> 3);
      rv[j] = s0 + ri < count;
      ro[j] = (uint32_t)work_spec(s, rv[j] ? s0 + ri : s0) * (uint32_t)(g.ldF / 4) + (lane & 7);
    }
    const float4 *fb4 = reinterpret_cast<const float4 *>(s.fbar);
    // lanes 0-31 stage basis rows 16-19 of the stage (row 32 + (lane >> 3))
    const float *bs = s.basis + (size_t)(16 + ((lane >> 3) & 3)) * g.ldF + 4 * (lane & 7);
    int c = cb;
    if (c + 32 <= ce) {
      float4 fv[4], fs, bv[kU];
      auto fetch = [&](int cc) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          fv[j] = rv[j] ? fb4[(size_t)ro[j] + cc / 4] : make_float4(0.f, 0.f, 0.f, 0.f);
        fs = lane < 32 ? *reinterpret_cast<const float4 *>(bs + cc) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int u = 0; u < kU; ++u) bv[u] = *reinterpret_cast<const float4 *>(b_ptr[0] + cc + 16 * u + 4 * kq);
      };
      fetch(c);
      for (; c + 32 <= ce; c += 32) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          *reinterpret_cast<float4 *>(stg + (8 * j + (lane >> 3)) * kSLd + 4 * (lane & 7)) = fv[j];
        if (lane < 32) *reinterpret_cast<float4 *>(stg + (32 + (lane >> 3)) * kSLd + 4 * (lane & 7)) = fs;
        float4 bcur[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) bcur[u] = bv[u];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (c + 64 <= ce) fetch(c + 32);  // next stage
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          float4 fa[2];
#pragma unroll
          for (int rt = 0; rt < 2; ++rt)
            fa[rt] = *reinterpret_cast<const float4 *>(stg + (16 * rt + i_row) * kSLd + 16 * u + 4 * kq);
          step16(fa, bcur[u]);
        }
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
          const float4 a4 = *reinterpret_cast<const float4 *>(stg + r4 * kSLd + 16 * hh + 4 * qq);
          const float4 w4 = *reinterpret_cast<const float4 *>(stg + (32 + j4) * kSLd + 16 * hh + 4 * qq);
          acc4[qq] = __builtin_amdgcn_mfma_f32_4x4x1f32(a4.x, w4.x, acc4[qq], 0, 0, 0);
          acc4[qq] = __builtin_amdgcn_mfma_f32_4x4x1f32(a4.y, w4.y, acc4[qq], 0, 0, 0);
          acc4[qq] = __builtin_amdgcn_mfma_f32_4x4x1f32(a4.z, w4.z, acc4[qq], 0, 0, 0);
          acc4[qq] = __builtin_amdgcn_mfma_f32_4x4x1f32(a4.w, w4.w, acc4[qq], 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
    for (; c < ce; c += 16) {  // a 16-column tail: lanes of half 1 add zeros
      float4 fa[2], bv[NG];
      load(IntC<0>{}, IntC<1>{}, c + 4 * kq, fa, bv);
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
        if (!row_ok[rt]) fa[rt] = make_float4(0.f, 0.f, 0.f, 0.f);
      step16(fa, bv[0]);
#pragma unroll
      for (int qq = 0; qq < 4; ++qq) {
        float4 a4 = *reinterpret_cast<const float4 *>(fb4row + c + 4 * qq);
        const float4 w4 = *reinterpret_cast<const float4 *>(b4 + c + 4 * qq);
        if (hh) a4 = make_float4(0.f, 0.f, 0.f, 0.f);
        acc4[qq] = __builtin_amdgcn_mfma_f32_4x4x1f32(a4.x, w4.x, acc4[qq], 0, 0, 0);
        acc4[qq] = __builtin_amdgcn_mfma_f32_4x4x1f32(a4.y, w4.y, acc4[qq], 0, 0, 0);
        acc4[qq] = __builtin_amdgcn_mfma_f32_4x4x1f32(a4.z, w4.z, acc4[qq], 0, 0, 0);
        acc4[qq] = __builtin_amdgcn_mfma_f32_4x4x1f32(a4.w, w4.w, acc4[qq], 0, 0, 0);
      }
    }
  } else {
    // an emulator class with zero weight and weight derivative for all 32
    // spectra (other Teff regimes) only ever multiplies its rows of
    // Phi-bar by zero: the 16-row groups that hold no other class's rows
    // are left out (classes are rows 0-19, 20-39, 40-59; groups 0-15,
    // 16-31, 32-47, 48-63)
    bool nz[kMaxClasses] = {false, false, false};
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      if (row_ok[rt]) {
        float w[kMaxClasses], dw[kMaxClasses];
        class_weights(g, s.u[(size_t)work_spec(s, s0 + 16 * rt + i_row) * kNP], w, dw);
#pragma unroll
        for (int q = 0; q < kMaxClasses; ++q) nz[q] = nz[q] || w[q] != 0.f || dw[q] != 0.f;
      }
    }
    int mask = 0;
#pragma unroll
    for (int q = 0; q < kMaxClasses; ++q) mask |= (__ballot(nz[q]) != 0) << q;
    switch (mask) {  // block uniform: all waves see the same 32 spectra
      case 1: run(IntC<0>{}, IntC<2>{}); break;
      case 2: run(IntC<1>{}, IntC<3>{}); break;
      case 4: run(IntC<2>{}, IntC<4>{}); break;
      case 3: run(IntC<0>{}, IntC<3>{}); break;
      case 6: run(IntC<1>{}, IntC<4>{}); break;
      default: run(IntC<0>{}, IntC<4>{}); break;
    }
  }
  __syncthreads();  // every wave is done with its stage: the buffer takes the partial sums
  if constexpr (NB == kNB) {
    // the blocks' sums; rows 16-19 have the two column halves in columns
    // 16-19 and 20-23
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        red[wave][16 * rt + 4 * kq + r][i_row] =
            (acc16[rt][r] + acc16[rt][4 + r]) + (acc16[rt][8 + r] + acc16[rt][12 + r]);
    const int g4 = (lane >> 2) & 7;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      red[wave][4 * g4 + r][16 + (lane & 3) + 4 * (lane >> 5)] =
          (acc4[0][r] + acc4[1][r]) + (acc4[2][r] + acc4[3][r]);
  } else {
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int q = 0; q < NG; ++q) red[wave][16 * rt + 4 * kq + r][16 * q + i_row] = acc[rt][q][r];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 32 * NB; e += 512) {
    const int i = e / NB, k = e - i * NB;
    float v;
    if (NB == kNB && k >= 16) {
      v = red[0][i][k] + red[0][i][k + 4];
#pragma unroll
      for (int w = 1; w < NWV; ++w) v += red[w][i][k] + red[w][i][k + 4];
    } else {
      v = red[0][i][k];
#pragma unroll
      for (int w = 1; w < NWV; ++w) v += red[w][i][k];
    }
    pb[i][k] = v;
  }
  __syncthreads();
  const int t = threadIdx.x;
  if (t < 32 && s0 + t < count)
    bwd_epilogue<NB>(g, s, adam, do_adam, grad_out, work_spec(s, s0 + t), pb[t]);
}

}  // namespace

hipError_t launch_interp_fwd(const Geometry &g, const State &s, int deriv_rows, int bf16x3,
                             hipStream_t st) {
  const int rows_per_spec = deriv_rows ? 4 : 1;
  const int rows = g.B * rows_per_spec;
  const int cols_per_block = 4 * 16 * kFwdTiles;
  const int col_blocks = (g.ldF + cols_per_block - 1) / cols_per_block;
  const int tiles = (rows + 15) / 16;
  int row_blocks = tiles;
  if (!fwd_one_tile(g, s)) {
    // workgroups for a work list of any length up to rows: it takes one tile
    // each up to two rounds of kFwdResident, then no more than one round
    // (BF16x3: then kFwdBf16Tiles each)
    int most = 2 * kFwdResident / col_blocks + 1;
    if (bf16x3) most = std::max(most, (tiles + kFwdBf16Tiles - 1) / kFwdBf16Tiles);
    row_blocks = std::min(tiles, most);
  }
  dim3 grid(col_blocks, row_blocks);
  // derivative rows are only formed for final evaluations: never skip those
  const int skip_done = deriv_rows ? 0 : 1;
  if (bf16x3)
    hipLaunchKernelGGL(k_interp_fwd_bf16, grid, dim3(256), 0, st, g, s, rows_per_spec, skip_done);
  else if (g.nb == kNB)
    hipLaunchKernelGGL(k_interp_fwd<kNB>, grid, dim3(256), 0, st, g, s, rows_per_spec, skip_done);
  else
    hipLaunchKernelGGL(k_interp_fwd<kNB * kMaxClasses>, grid, dim3(256), 0, st, g, s,
                       rows_per_spec, skip_done);
  return hipGetLastError();
}

hipError_t launch_interp_bwd(const Geometry &g, const State &s, const AdamCfg *adam,
                             float *grad_out, int bf16x3, hipStream_t st) {
  AdamCfg a = adam ? *adam : AdamCfg{0.f, 0.f, 0.f, 0.f, 0, 0.f};
  const dim3 grid((g.B + 15) / 16);
  if (bf16x3)
    hipLaunchKernelGGL(k_interp_bwd_bf16, grid, dim3(256), 0, st, g, s, a, adam ? 1 : 0, grad_out);
  else if (g.nb == kNB)
    hipLaunchKernelGGL((k_interp_bwd<kNB>), dim3((g.B + 31) / 32), dim3(512), 0, st, g, s, a,
                       adam ? 1 : 0, grad_out);
  else
    hipLaunchKernelGGL((k_interp_bwd<kNB * kMaxClasses>), dim3((g.B + 31) / 32), dim3(512), 0,
                       st, g, s, a, adam ? 1 : 0, grad_out);
  return hipGetLastError();
}

hipError_t launch_split_basis(const Geometry &g, const State &s, hipStream_t st) {
  hipLaunchKernelGGL(k_split_basis, dim3((g.ldF + 255) / 256, kNB + 4), dim3(256), 0, st, g, s);
  return hipGetLastError();
}

}  // namespace lasp
