// Dense near-field blocks at many frequencies at once.
//
// The entries of every inadmissible block are written for F frequencies into
// out[f * stride + near_off[q] + e] (e column-major inside the block).  Two
// passes keep the waves uniform:
//   near_far_tier: one thread per entry, NEAR_SPLIT workgroups per block (a
//     few hundred blocks of 64 x 64 entries would not fill the chip); entries of
//     the far tier (7-point rule); self and near-tier entries are skipped;
//   near_sing: one wave per self/near-tier entry (polar-coordinate self rule or
//     112-point rule).
// Both evaluate a pair's geometry once and its frequencies by the series of
// series.h (the far tier in double point by point), bound by float64 issue and,
// in float, the stores (3648 triangles at 129 frequencies, complex64: near_sing
// 24.5 -> 2.7 ms, near_far_tier 12.1 -> 5.4 ms against a sum per point and
// frequency).
// DLP: the double layer's entries (normal derivative in y; self entries 0).
// The list of self/near-tier entries is built once with the block tree.
#pragma once
#include "series.h"

namespace gcq {

struct SingEntry {
  int64_t off;   // element offset inside one frequency's near storage
  int pi, pj;    // internal positions
};

constexpr int NEAR_SPLIT = 4;
template <typename T, bool DLP = false>
__global__ void __launch_bounds__(FAR_THREADS) near_far_tier(Tab tab, const int* __restrict__ blk,
                                                     const int* __restrict__ near_ids,
                                                     const int64_t* __restrict__ near_off,
                                                     int q0, int q1, int64_t base0,
                                                     const double2* __restrict__ sig, int F, double smax,
                                                     cpx<T>* __restrict__ out, int64_t stride) {
  __shared__ double pts[far_pts<T>()];
  for (int q = q0 + blockIdx.x; q < q1; q += gridDim.x) {
    const int id = near_ids[q];
    const int rb = blk[5 * id], m = blk[5 * id + 1] - rb, cb = blk[5 * id + 2];
    const int n = blk[5 * id + 3] - cb;
    const int64_t base = near_off[q] - base0;
    // (every lane takes part in the wave's maximum; gridDim.y workgroups share a block)
    for (int e0 = blockIdx.y * FAR_THREADS; e0 < m * n; e0 += gridDim.y * FAR_THREADS) {
      const int e = e0 + threadIdx.x, ec = min(e, m * n - 1);
      const int pi = rb + ec % m, pj = cb + ec / m;
      const bool ok = e < m * n && pi != pj && !is_near(tab, pi, pj);
      cpx<T>* o = out + base + e;
      far_pair<T, DLP>(tab, pi, pj, ok, sig, 0, F, 1, smax, sizeof(T) == 4 ? pts + threadIdx.x : pts,
                       [&](int f, cpx<T> v) { o[int64_t(f) * stride] = v; });
    }
  }
}

template <typename T, bool DLP = false>
__global__ void __launch_bounds__(256) near_sing(Tab tab, const SingEntry* __restrict__ list,
                                                 int64_t s0, int64_t s1, int64_t base0,
                                                 const double2* __restrict__ sig, int F, double smax,
                                                 cpx<T>* __restrict__ out, int64_t stride) {
  __shared__ double lds[4 * SERIES_LDS];
  const int w = uni(threadIdx.x / WAVE);
  for (int64_t a = s0 + int64_t(blockIdx.x) * 4 + w; a < s1; a += int64_t(gridDim.x) * 4) {
    const SingEntry se = list[a];
    cpx<T>* o = out + se.off - base0;
    near_pair<T, DLP>(tab, uni(se.pi), uni(se.pj), sig, F, smax, lds + w * SERIES_LDS,
                      [&](int f, cpx<T> v) { o[int64_t(f) * stride] = v; });
  }
}

}  // namespace gcq
