// Continuum moments of one lane's pixels (Eq. 6), shared by the fused pass
// and the covariance kernel.
#pragma once

#include "lasp_internal.h"

// Every fused multiply-add is written out (the callers' variants then agree
// bit for bit).
#pragma clang fp contract(off)

namespace lasp {

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
// interpolation error 2 (a / 2)^7 |p^(7)| / 7!, a = 16 / P, with the seventh
// derivative of a degree-n polynomial bounded by one, prod_{k < 7} (n^2 - k^2)
// / (2 k + 1) (Markov).  Degree 10: 1,872 pixels and more, 8: 1,176, 6: 632,
// 4: 240; shorter rows sum over the pixels.  (Six nodes would serve 3,684
// pixels and more at degree 10; the step's pass measured 0.290 ms with six,
// 0.293 with seven and 0.321 with both in one kernel, 16,384 x 3,900.)
inline bool moment_nodes_hold(int nd, int P) {
  const double n = 2.0 * (nd - 1), a = 16.0 / (double)P;
  double b = 2.0;
  for (int k = 0; k < kNodes; ++k) b *= (n * n - (double)k * k) / (2.0 * k + 1.0) / (k + 1.0) * 0.5 * a;
  return b <= 1e-7;
}

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

}  // namespace lasp
