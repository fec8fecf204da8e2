// Products with the 3D-ACA form (eq. product):
//   PER_FREQUENCY  Y[k] = sum_b sum_d f_{b,d}[k] H_{b,d} X[k][J_b]
//   WEIGHTED_SUM   y    = sum_b sum_d H_{b,d} (sum_k f_{b,d}[k] X[k][J_b])
// with the conjugate-partner rule for columns whose frequency is represented by
// its conjugate.
#include <algorithm>
#include <cstring>

#include <type_traits>

#include "internal.h"
#include "matvec.h"

namespace gcq {

template <typename TI, typename TO>
__global__ void perm_in3(const cpx<TI>* __restrict__ X, cpx<TO>* __restrict__ Xp,
                         const int* __restrict__ perm, const int* __restrict__ conjflag, int n,
                         int L) {
  const int64_t total = int64_t(n) * L;
  for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total;
       e += int64_t(gridDim.x) * blockDim.x) {
    const int k = int(e / n), p = int(e % n);
    cpx<TI> v = X[int64_t(k) * n + perm[p]];
    Xp[e] = {TO(v.re), conjflag[k] ? TO(-v.im) : TO(v.im)};
  }
}

template <typename TI, typename TO>
__global__ void perm_out3(const cpx<TI>* __restrict__ Yp, cpx<TO>* __restrict__ Y,
                          const int* __restrict__ perm, const int* __restrict__ conjflag, int n,
                          int L) {
  const int64_t total = int64_t(n) * L;
  for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total;
       e += int64_t(gridDim.x) * blockDim.x) {
    const int k = int(e / n), p = int(e % n);
    cpx<TI> v = Yp[e];
    Y[int64_t(k) * n + perm[p]] = {TO(v.re), conjflag[k] ? TO(-v.im) : TO(v.im)};
  }
}

template <typename T>
__global__ void zero3(cpx<T>* p, int64_t n) {
  for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < n;
       e += int64_t(gridDim.x) * blockDim.x)
    p[e] = {T(0), T(0)};
}

// Xp[p][k] = X[k][perm[p]] (frequency fastest), conjugated for columns applied
// through their conjugate partner, and Yp = 0; and the inverse for the result
template <typename TI, typename TO>
__global__ void perm_in_t(const cpx<TI>* __restrict__ X, cpx<TO>* __restrict__ Xp, cpx<TO>* __restrict__ Yp,
                          const int* __restrict__ perm, const int* __restrict__ conjflag, int n,
                          int L) {
  const int64_t total = int64_t(n) * L;
  for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total;
       e += int64_t(gridDim.x) * blockDim.x) {
    const int p = int(e / L), k = int(e % L);
    cpx<TI> v = X[int64_t(k) * n + perm[p]];
    Xp[e] = {TO(v.re), conjflag[k] ? TO(-v.im) : TO(v.im)};
    Yp[e] = {TO(0), TO(0)};
  }
}

template <typename TI, typename TO>
__global__ void perm_out_t(const cpx<TI>* __restrict__ Yp, cpx<TO>* __restrict__ Y,
                           const int* __restrict__ perm, const int* __restrict__ conjflag, int n,
                           int L) {
  const int64_t total = int64_t(n) * L;
  for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total;
       e += int64_t(gridDim.x) * blockDim.x) {
    const int p = int(e / L), k = int(e % L);
    cpx<TI> v = Yp[e];
    Y[int64_t(k) * n + perm[p]] = {TO(v.re), conjflag[k] ? TO(-v.im) : TO(v.im)};
  }
}

// ---- per-frequency product on the matrix cores ----------------------------------
// Per far block (R stacked columns, Ubar m x R, Vbar n x R, column-major, the
// block's stack contiguous): T = Vbar^H X_J, T' = F o T with F[c][k] = f_c[rep(k)],
// Y_I += Ubar T'.  Per near block: Y_I += sum_d f_d[rep(k)] (D_d X_J)[:, k].
//
// Tiles of 16 rows by 16 frequency columns, four contraction values a step
// (v_mfma_f32_16x16x4f32, v_mfma_f64_16x16x4f64: A[i][k] in lane i + 16 k, B[k][j] in
// lane j + 16 k): leaves of 40 rows pad to 48, where 32-row tiles pad to 64, at the
// same rate.  A wave multiplies two column tiles, so that an operator value
// serves both.  Operator values are loaded a term (near) or KU steps
// (far) ahead, which memory latency takes at two waves a SIMD; indices beyond a block are clamped, against zeros on the other side of the product.
//   near: a wave per (block, 16 rows, 16 CT columns), NEAR_XS steps of X_J in
//     registers over the block's terms (X_J was re-read per term), wider blocks
//     in several pieces.  CT = 1 where there are too few waves for the chip.
//   far: a workgroup of four waves per (block, FC columns), T' of up to MM_CC
//     stacked columns in LDS, larger stacks MM_CC at a time.
// The workgroups of one block's column chunks have numbers 8 apart, so that they
// run on one XCD and share the block in its L2.  Bound by the matrix cores and,
// on small partitions, by latency.  5120-triangle sphere, 64 frequencies: 0.90 ms
// in complex64 (1.36 with 32-row tiles, one workgroup a block), 1.4 ms in
// complex128 (8.6 on the vector units).  Accumulation into Yp with atomics.
typedef float mm_f4 __attribute__((ext_vector_type(4)));
typedef double mm_d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ mm_f4 mm(float a, float b, mm_f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ mm_d4 mm(double a, double b, mm_d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

template <typename T>
struct Mm;
template <>
struct Mm<float> {
  static constexpr int NEAR_XS = 16;   // steps of X_J held: 64 columns
  static constexpr int FC = 64;        // far: frequency columns of a workgroup
  static constexpr int KU = 8;         // far: steps whose operands are loaded together, ahead of their products
  // complex accumulator in Gauss's three products: k1 += (a_r + a_i) b_r,
  // k2 += a_r (b_i - b_r), k3 += a_i (b_r + b_i); Re = k1 - k3, Im = k1 + k2
  mm_f4 k1 = {0.f, 0.f, 0.f, 0.f}, k2 = k1, k3 = k1;
  __device__ __forceinline__ void step(cpx<float> a, cpx<float> b) {
    k1 = mm(a.re + a.im, b.re, k1);
    k2 = mm(a.re, b.im - b.re, k2);
    k3 = mm(a.im, b.re + b.im, k3);
  }
  __device__ __forceinline__ cpx<float> get(int r) const { return {k1[r] - k3[r], k1[r] + k2[r]}; }
  static __device__ __forceinline__ int row(int r, int q) { return 4 * q + r; }   // of element r, lane group q
};
template <>
struct Mm<double> {
  static constexpr int NEAR_XS = 10;
  static constexpr int FC = 32;
  static constexpr int KU = 4;
  mm_d4 re = {0.0, 0.0, 0.0, 0.0}, im = re;
  __device__ __forceinline__ void step(cpx<double> a, cpx<double> b) {
    re = mm(a.re, b.re, re);
    im = mm(a.re, b.im, im);
    re = mm(-a.im, b.im, re);
    im = mm(a.im, b.re, im);
  }
  __device__ __forceinline__ cpx<double> get(int r) const { return {re[r], im[r]}; }
  static __device__ __forceinline__ int row(int r, int q) { return 4 * r + q; }
};

constexpr int MM_CC = 128;   // stacked columns of T' in LDS

template <typename T>
__device__ __forceinline__ void add_rows(cpx<T>* __restrict__ Yp, int rb, int m, int i0, int q, int L, int k,
                                         const cpx<T> (&v)[4]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = i0 + Mm<T>::row(r, q);
    if (i < m) {
      cpx<T>* y = Yp + int64_t(rb + i) * L + k;
      atomicAdd(&y->re, v[r].re);
      atomicAdd(&y->im, v[r].im);
    }
  }
}

// far: workgroups [0, wfar), near: the others, a task (block, row tile, column
// chunk) per wave
template <typename T, int CT>
__global__ void __launch_bounds__(256, 2) perfreq_mm(
    const int* __restrict__ blk, const int* __restrict__ farlist, int nfar, int wfar,
    const int2* __restrict__ neartask, int nnear, const int* __restrict__ bterm, const int64_t* __restrict__ toff,
    const int64_t* __restrict__ tfoff, const int64_t* __restrict__ cols, const int* __restrict__ bcol,
    const cpx<T>* __restrict__ pool, const int* __restrict__ colpos, int L, const cpx<T>* __restrict__ Xp,
    cpx<T>* __restrict__ Yp) {
  constexpr int FC = Mm<T>::FC, KU = Mm<T>::KU, TS = FC + 8;   // (row stride of T': the four rows a read touches in other banks)
  __shared__ cpx<T> Ts[MM_CC * TS];
  const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const cpx<T> zero = {T(0), T(0)};
  if (int(blockIdx.x) >= wfar) {
    constexpr int XS = Mm<T>::NEAR_XS;
    // task numbers: column chunks of four tasks 8 workgroups apart
    const int nkc = (L + 16 * CT - 1) / (16 * CT);
    const int id = blockIdx.x - wfar, loc = id >> 3;
    const int ti = ((loc / nkc) * 8 + (id & 7)) * 4 + w, k0 = (loc % nkc) * 16 * CT;
    if (ti >= nnear) return;
    const int2 task = neartask[ti];
    const int b = task.x, i0 = task.y;
    const int rb = blk[5 * b], m = blk[5 * b + 1] - rb, cb = blk[5 * b + 2], n = blk[5 * b + 3] - cb;
    const int d0 = bterm[b], d1 = bterm[b + 1];
    const int ia = min(i0 + l16, m - 1);
    bool kin[CT];
    int kp[CT];
#pragma unroll
    for (int u = 0; u < CT; ++u) {
      kin[u] = k0 + 16 * u + l16 < L;
      kp[u] = kin[u] ? colpos[k0 + 16 * u + l16] : 0;
    }
    cpx<T> y[CT][4];
#pragma unroll
    for (int u = 0; u < CT; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) y[u][r] = zero;
    for (int j0 = 0; j0 < n; j0 += 4 * XS) {
      const int jn = min(4 * XS, n - j0);
      cpx<T> x[XS][CT];
#pragma unroll
      for (int s = 0; s < XS; ++s)
#pragma unroll
        for (int u = 0; u < CT; ++u) {
          const int j = 4 * s + q;
          x[s][u] = (j < jn && kin[u]) ? Xp[int64_t(cb + j0 + j) * L + k0 + 16 * u + l16] : zero;
        }
      // a[s]: step s of the current term, replaced by the next term's as it is used
      const cpx<T>* D = pool + toff[d0] + int64_t(j0) * m + ia;
      cpx<T> a[XS];
#pragma unroll
      for (int s = 0; s < XS; ++s) a[s] = D[min(4 * s + q, jn - 1) * m];
      for (int d = d0; d < d1; ++d) {
        const cpx<T>* Dn = d + 1 < d1 ? pool + toff[d + 1] + int64_t(j0) * m + ia : D;
        cpx<T> f[CT];
#pragma unroll
        for (int u = 0; u < CT; ++u) f[u] = pool[tfoff[d] + kp[u]];
        Mm<T> t[CT];
#pragma unroll
        for (int s = 0; s < XS; ++s) {
          if (4 * s >= jn) break;
          const cpx<T> c = a[s];
          a[s] = Dn[min(4 * s + q, jn - 1) * m];
#pragma unroll
          for (int u = 0; u < CT; ++u) t[u].step(c, x[s][u]);
        }
        D = Dn;
#pragma unroll
        for (int u = 0; u < CT; ++u)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const cpx<T> p = cmul(f[u], t[u].get(r));
            y[u][r].re += p.re;
            y[u][r].im += p.im;
          }
      }
    }
#pragma unroll
    for (int u = 0; u < CT; ++u)
      if (kin[u]) add_rows<T>(Yp, rb, m, i0, q, L, k0 + 16 * u + l16, y[u]);
    return;
  }
  const int nkc = (L + FC - 1) / FC;
  const int loc = blockIdx.x >> 3, fi = (loc / nkc) * 8 + (blockIdx.x & 7), kc = (loc % nkc) * FC;
  if (fi >= nfar) return;
  const int b = farlist[fi];
  const int rb = blk[5 * b], m = blk[5 * b + 1] - rb, cb = blk[5 * b + 2], n = blk[5 * b + 3] - cb;
  const int c0b = bcol[b], R = bcol[b + 1] - c0b;
  if (R == 0) return;
  const cpx<T>* Ust = pool + cols[3 * c0b];
  const cpx<T>* Vst = pool + cols[3 * c0b + 1];
  const int halves = min(FC, L - kc) > 32 ? 2 : 1;   // 32-column halves that hold a column
  for (int cc = 0; cc < R; cc += MM_CC) {
    const int cn = min(MM_CC, R - cc), ct = (cn + 15) >> 4;
    if (cc > 0) __syncthreads();   // the last chunk's T' is read
    // T' = F o (Vbar^H X_J) for stacked columns cc .. cc + cn
    for (int tile = w; tile < ct * halves; tile += 4) {
      const int ti = tile / halves, kb = kc + (tile % halves) * 32;
      bool kin[2];
      const cpx<T>* xk[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        kin[u] = kb + 16 * u + l16 < L;
        xk[u] = Xp + int64_t(cb) * L + (kin[u] ? kb + 16 * u + l16 : 0);
      }
      const cpx<T>* Vc = Vst + int64_t(min(cc + ti * 16 + l16, R - 1)) * n;
      Mm<T> t[2];
      cpx<T> a[KU], x[KU][2];
      auto load = [&](int j0) {
#pragma unroll
        for (int v = 0; v < KU; ++v) {
          const int j = j0 + 4 * v + q, jc = min(j, n - 1);
          a[v] = Vc[jc];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const cpx<T> xx = xk[u][int64_t(jc) * L];
            x[v][u] = (j < n && kin[u]) ? xx : zero;
          }
        }
      };
      load(0);
      for (int j0 = 0; j0 < n; j0 += 4 * KU) {
        cpx<T> c[KU], xc[KU][2];
#pragma unroll
        for (int v = 0; v < KU; ++v) {
          c[v] = {a[v].re, -a[v].im};   // conj(v)
          xc[v][0] = x[v][0];
          xc[v][1] = x[v][1];
        }
        if (j0 + 4 * KU < n) load(j0 + 4 * KU);
#pragma unroll
        for (int v = 0; v < KU; ++v)
#pragma unroll
          for (int u = 0; u < 2; ++u) t[u].step(c[v], xc[v][u]);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int kp = kin[u] ? colpos[kb + 16 * u + l16] : 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int cl = ti * 16 + Mm<T>::row(r, q);   // local stacked column
          cpx<T> v = zero;
          if (cl < cn && kin[u]) v = cmul(pool[cols[3 * (c0b + cc + cl) + 2] + kp], t[u].get(r));
          Ts[cl * TS + kb - kc + 16 * u + l16] = v;
        }
      }
    }
    __syncthreads();
    // Y_I += Ubar[:, cc .. cc + cn] T'
    const int mt = (m + 15) >> 4;
    for (int tile = w; tile < mt * halves; tile += 4) {
      const int i0 = (tile / halves) * 16, kb = kc + (tile % halves) * 32;
      const cpx<T>* Ui = Ust + int64_t(cc) * m + min(i0 + l16, m - 1);
      Mm<T> t[2];
      cpx<T> a[KU];
#pragma unroll
      for (int v = 0; v < KU; ++v) a[v] = Ui[int64_t(min(4 * v + q, cn - 1)) * m];
      for (int c2 = 0; c2 < cn; c2 += 4 * KU) {
        cpx<T> c[KU];
#pragma unroll
        for (int v = 0; v < KU; ++v) {
          c[v] = a[v];
          a[v] = Ui[int64_t(min(c2 + 4 * KU + 4 * v + q, cn - 1)) * m];
        }
#pragma unroll
        for (int v = 0; v < KU; ++v)
#pragma unroll
          for (int u = 0; u < 2; ++u)
            if (c2 + 4 * v < 16 * ct) t[u].step(c[v], Ts[(c2 + 4 * v + q) * TS + kb - kc + 16 * u + l16]);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int k = kb + 16 * u + l16;
        const cpx<T> v[4] = {t[u].get(0), t[u].get(1), t[u].get(2), t[u].get(3)};
        if (k < L) add_rows<T>(Yp, rb, m, i0, q, L, k, v);
      }
    }
  }
}

// eq. product: a workgroup of NT threads per block, up to WS_D terms of it at a
// time.  Per piece of WS_J columns the frequency sums w1_d (plain columns) and
// w2_d (conjugate-represented columns, conjugated input) of all those terms form
// in one pass over X (the fibers staged in LDS, the frequencies dealt to the
// threads that a narrow block leaves over); then y_I += sum_d H_d w1_d +
// conj(H_d w2_d), a far block through its stacked factors: t = Vbar^H w, 16
// lanes a column, and y = Ubar t, a thread a row.  Bound by the stored slices'
// bytes, each read once (one wave per block and one term at a time, which read X
// anew for every term, took 11.4 ms on the 20480-triangle sphere at 64
// frequencies; now 3.6 with four waves and eight terms).  Accumulation into y with
// atomics.
template <typename T, int NT, int WS_D, int WS_J, int WS_K>
__global__ void __launch_bounds__(NT) wsum_kernel(
    const int* __restrict__ blk, const int* __restrict__ order, int nblocks, const int* __restrict__ bterm,
    const int* __restrict__ trank, const int64_t* __restrict__ toff,
    const int64_t* __restrict__ tvoff, const int64_t* __restrict__ tfoff,
    const cpx<T>* __restrict__ pool, const int* __restrict__ colpos,
    const int* __restrict__ conjf, int L, int n,
    const cpx<T>* __restrict__ X, cpx<T>* __restrict__ ybuf) {
  constexpr int WS_R = WS_D * 64;
  __shared__ cpx<T> ws[2][WS_D][WS_J];
  __shared__ cpx<T> fs[WS_D][WS_K];
  __shared__ cpx<T> ts[2][WS_R];
  __shared__ cpx<T> red[NT];
  __shared__ unsigned char cterm[WS_R];
  __shared__ unsigned char cj[WS_K];
  const int tid = threadIdx.x;
  for (int ob = blockIdx.x; ob < nblocks; ob += gridDim.x) {
    const int b = order[ob];   // blocks with terms, most work first
    const int rb = blk[5 * b], m = blk[5 * b + 1] - rb, cb = blk[5 * b + 2], nn = blk[5 * b + 3] - cb;
    const bool far = trank[bterm[b]] >= 0;
    const int jt = nn <= 64 ? 64 : WS_J, kg = tid / jt, nkg = NT / jt, jl = tid % jt;
    const int it = min(NT, m <= 64 ? 64 : m <= 128 ? 128 : 256), ig = tid / it, nig = NT / it;
    for (int d0 = bterm[b]; d0 < bterm[b + 1]; d0 += WS_D) {
      const int nd = min(WS_D, bterm[b + 1] - d0);
      int R = 0;
      __syncthreads();   // the last piece's readers are done
      if (far)
        for (int d = 0; d < nd; ++d) {
          const int r = trank[d0 + d];
          for (int c = tid; c < r; c += NT) cterm[R + c] = (unsigned char)d;
          R += r;
        }
      for (int j0 = 0; j0 < nn; j0 += WS_J) {
        const int jn = min(WS_J, nn - j0);
        cpx<T> a1[WS_D], a2[WS_D];
#pragma unroll
        for (int d = 0; d < WS_D; ++d) a1[d] = a2[d] = {T(0), T(0)};
        for (int k0 = 0; k0 < L; k0 += WS_K) {
          const int kn = min(WS_K, L - k0);
          __syncthreads();
          for (int e = tid; e < WS_D * WS_K; e += NT) {
            const int d = e / WS_K, k = e % WS_K;
            fs[d][k] = (d < nd && k < kn) ? pool[tfoff[d0 + d] + colpos[k0 + k]] : cpx<T>{T(0), T(0)};
          }
          if (tid < kn) cj[tid] = (unsigned char)conjf[k0 + tid];
          __syncthreads();
          if (jl < jn)
            for (int k = kg; k < kn; k += nkg) {
              const cpx<T> x = X[int64_t(k0 + k) * n + cb + j0 + jl];   // cluster order, not conjugated
              if (uni(cj[k])) {
#pragma unroll
                for (int d = 0; d < WS_D; ++d) {
                  const cpx<T> f = fs[d][k];
                  a2[d].re += f.re * x.re + f.im * x.im;   // f conj(x)
                  a2[d].im += f.im * x.re - f.re * x.im;
                }
              } else {
#pragma unroll
                for (int d = 0; d < WS_D; ++d) {
                  const cpx<T> f = fs[d][k];
                  a1[d].re += f.re * x.re - f.im * x.im;
                  a1[d].im += f.re * x.im + f.im * x.re;
                }
              }
            }
        }
        for (int g = 0; g < nkg; ++g) {   // the frequency groups' sums, in group order
          if (kg == g)
#pragma unroll
            for (int d = 0; d < WS_D; ++d) {
              const cpx<T> o1 = g ? ws[0][d][jl] : cpx<T>{T(0), T(0)}, o2 = g ? ws[1][d][jl] : cpx<T>{T(0), T(0)};
              ws[0][d][jl] = {o1.re + a1[d].re, o1.im + a1[d].im};
              ws[1][d][jl] = {o2.re + a2[d].re, o2.im + a2[d].im};
            }
          __syncthreads();
        }
        if (far) {
          // t[c] over this piece of columns, 16 lanes a column
          const cpx<T>* V = pool + tvoff[d0] + j0;
          const int q = tid & 15;
          for (int c = tid >> 4; c < R; c += NT / 16) {
            const int d = cterm[c];
            const cpx<T>* Vc = V + int64_t(c) * nn;
            T r1 = 0, i1 = 0, r2 = 0, i2 = 0;
            for (int j = q; j < jn; j += 16) {
              const cpx<T> v = Vc[j], p1 = cmulc(v, ws[0][d][j]), p2 = cmulc(v, ws[1][d][j]);
              r1 += p1.re; i1 += p1.im;
              r2 += p2.re; i2 += p2.im;
            }
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) {
              r1 += __shfl_xor(r1, o, WAVE);
              i1 += __shfl_xor(i1, o, WAVE);
              r2 += __shfl_xor(r2, o, WAVE);
              i2 += __shfl_xor(i2, o, WAVE);
            }
            if (q == 0) {
              const cpx<T> o1 = j0 ? ts[0][c] : cpx<T>{T(0), T(0)}, o2 = j0 ? ts[1][c] : cpx<T>{T(0), T(0)};
              ts[0][c] = {o1.re + r1, o1.im + i1};
              ts[1][c] = {o2.re + r2, o2.im + i2};
            }
          }
          if (j0 + WS_J < nn) continue;
          __syncthreads();
        }
        // rows: far from all columns' t, near from this piece's w
        for (int i0 = 0; i0 < m; i0 += it) {
          const int i = i0 + tid % it;
          T re = 0, im = 0;
          if (i < m) {
            if (far) {
              const cpx<T>* U = pool + toff[d0] + i;
              T r2 = 0, i2 = 0;
              for (int c = ig; c < R; c += nig) {
                const cpx<T> u = U[int64_t(c) * m], p1 = cmul(u, ts[0][c]), p2 = cmul(u, ts[1][c]);
                re += p1.re; im += p1.im;
                r2 += p2.re; i2 += p2.im;
              }
              re += r2;
              im -= i2;
            } else {
              T r2 = 0, i2 = 0;
              for (int d = 0; d < nd; ++d) {
                const cpx<T>* D = pool + toff[d0 + d] + int64_t(j0) * m + i;
                for (int j = ig; j < jn; j += nig) {
                  const cpx<T> h = D[int64_t(j) * m], p1 = cmul(h, ws[0][d][j]), p2 = cmul(h, ws[1][d][j]);
                  re += p1.re; im += p1.im;
                  r2 += p2.re; i2 += p2.im;
                }
              }
              re += r2;
              im -= i2;
            }
          }
          if (nig > 1) {
            red[tid] = {re, im};
            __syncthreads();
            if (ig == 0)
              for (int g = 1; g < nig; ++g) {
                re += red[g * it + tid].re;
                im += red[g * it + tid].im;
              }
            __syncthreads();
          }
          if (ig == 0 && i < m) {
            atomicAdd(&ybuf[rb + i].re, re);
            atomicAdd(&ybuf[rb + i].im, im);
          }
        }
      }
    }
  }
}

// the kernels of the per-frequency product on stream st (no allocation, no
// host transfer: a capturable sequence)
template <typename T>
static void enqueue_perfreq(gcq_context* ctx, hipStream_t st, int precision, const void* X, void* Y) {
  Faces3D& F = ctx->F;
  const int n = ctx->n, L = ctx->L;
  const int64_t nl = int64_t(n) * L;
  cpx<T>* Xp = F.pxy.as<cpx<T>>();
  cpx<T>* Yp = Xp + nl;
  const int* d_colpos = F.pmeta.as<int>();
  const int* d_conj = d_colpos + L;
  const int* perm = ctx->d_perm.as<int>();
  const int g = int(std::min<int64_t>((nl + 255) / 256, 4096));
  if (precision == GCQ_C128)
    hipLaunchKernelGGL((perm_in_t<double, T>), dim3(g), dim3(256), 0, st, (const cpx<double>*)X, Xp, Yp,
                       perm, d_conj, n, L);
  else
    hipLaunchKernelGGL((perm_in_t<float, T>), dim3(g), dim3(256), 0, st, (const cpx<float>*)X, Xp, Yp,
                       perm, d_conj, n, L);
  // two column tiles a wave, one where the near blocks would not give every SIMD
  // two waves
  auto go = [&](auto ct) {
    constexpr int CT = decltype(ct)::value;
    const int kf = (L + Mm<T>::FC - 1) / Mm<T>::FC, kn = (L + 16 * CT - 1) / (16 * CT);
    const int wfar = (F.n_far + 7) / 8 * 8 * kf, wnear = (F.n_neartask + 31) / 32 * 8 * kn;
    if (wfar + wnear > 0)
      hipLaunchKernelGGL((perfreq_mm<T, CT>), dim3(wfar + wnear), dim3(256), 0, st, ctx->d_blk.as<int>(),
                         F.d_farlist.as<int>(), F.n_far, wfar, F.d_neartask.as<int2>(), F.n_neartask,
                         F.d_bterm.as<int>(), F.d_toff.as<int64_t>(), F.d_tfoff.as<int64_t>(),
                         F.d_cols.as<int64_t>(), F.d_bcol.as<int>(), F.slices.as<cpx<T>>(), d_colpos, L, Xp, Yp);
  };
  if (int64_t(F.n_neartask) * ((L + 31) / 32) < int64_t(ctx->cus) * 8)
    go(std::integral_constant<int, 1>());
  else
    go(std::integral_constant<int, 2>());
  if (precision == GCQ_C128)
    hipLaunchKernelGGL((perm_out_t<T, double>), dim3(g), dim3(256), 0, st, Yp, (cpx<double>*)Y, perm,
                       d_conj, n, L);
  else
    hipLaunchKernelGGL((perm_out_t<T, float>), dim3(g), dim3(256), 0, st, Yp, (cpx<float>*)Y, perm,
                       d_conj, n, L);
}

// the product's buffers and frequency tables (once per operator)
static int product_setup(gcq_context* ctx, size_t need) {
  Faces3D& F = ctx->F;
  const int L = ctx->L;
  if (F.pxy.bytes < need || !F.meta_valid) {
    F.graphs.clear();   // captured graphs refer to the old buffers and tables
    GCQ_TRY(F.pxy.ensure(need));
    std::vector<int> meta(2 * L);
    for (int k = 0; k < L; ++k) {
      meta[k] = ctx->kpos[k];
      meta[L + k] = ctx->conj[k];
    }
    GCQ_TRY(upload(F.pmeta, meta, ctx->stream));
    GCQ_HIP(hipStreamSynchronize(ctx->stream));
    F.meta_valid = true;
  }
  return GCQ_OK;
}

template <typename T>
static int compressed_impl(gcq_context* ctx, int mode, int precision, const void* X, void* Y) {
  Faces3D& F = ctx->F;
  hipStream_t st = ctx->stream;
  const int n = ctx->n, L = ctx->L, nb = int(ctx->blocks.size());
  if (mode == GCQ_PER_FREQUENCY) {
    const bool bf = precision == GCQ_C64_SPLIT_BF16;
    if (bf) GCQ_TRY(bf16_setup(ctx));
    GCQ_TRY(product_setup(ctx, bf ? bf16_buffer_bytes(ctx) : size_t(2) * n * L * sizeof(cpx<T>)));
    auto enqueue = [&](hipStream_t s) {
      if (bf)
        enqueue_perfreq_bf16(ctx, s, X, Y);
      else
        enqueue_perfreq<T>(ctx, s, precision, X, Y);
    };
    if (ctx->tune.product_graph) {
      hipGraphExec_t exec = nullptr;
      for (auto& x : F.graphs.e)
        if (x.X == X && x.Y == Y && x.precision == precision) exec = x.exec;
      if (!exec) {
        if (!F.graphs.cap) GCQ_HIP(hipStreamCreateWithFlags(&F.graphs.cap, hipStreamNonBlocking));
        hipGraph_t graph = nullptr;
        GCQ_HIP(hipStreamBeginCapture(F.graphs.cap, hipStreamCaptureModeThreadLocal));
        enqueue(F.graphs.cap);
        const hipError_t ce = hipGetLastError();
        GCQ_HIP(hipStreamEndCapture(F.graphs.cap, &graph));
        if (ce != hipSuccess) {
          (void)hipGraphDestroy(graph);
          return fail(GCQ_ERR_HIP, "capture of the product failed: %s", hipGetErrorString(ce));
        }
        const hipError_t ie = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (ie != hipSuccess) return fail(GCQ_ERR_HIP, "graph instantiation failed: %s", hipGetErrorString(ie));
        if (F.graphs.e.size() >= 8) {   // keep the most recent few
          (void)hipGraphExecDestroy(F.graphs.e.front().exec);
          F.graphs.e.erase(F.graphs.e.begin());
        }
        F.graphs.e.push_back({X, Y, precision, exec});
      }
      GCQ_TRY(timed_begin(ctx));
      GCQ_HIP(hipGraphLaunch(exec, st));
    } else {
      GCQ_TRY(timed_begin(ctx));
      enqueue(st);
    }
    GCQ_HIP(hipGetLastError());
    timed_end(ctx, "matvec_perfreq");
    return GCQ_OK;
  }
  std::vector<int> meta(2 * L);
  for (int k = 0; k < L; ++k) {
    meta[k] = ctx->kpos[k];
    meta[L + k] = ctx->conj[k];
  }
  GCQ_TRY(upload(ctx->scratchC, meta, st));
  const int* d_colpos = ctx->scratchC.as<int>();
  const int* d_conj = d_colpos + L;
  const int64_t nl = int64_t(n) * L;
  const int nmv = F.n_mvblocks;
  const int wgrid = std::max(1, std::min(nmv, ctx->cus * 32));
  GCQ_TRY(ctx->scratchB.ensure(size_t(nl + n) * sizeof(cpx<T>)));
  cpx<T>* Xp = ctx->scratchB.as<cpx<T>>();
  cpx<T>* Yp = Xp + nl;
  const int g = 4096;
  const int* perm = ctx->d_perm.as<int>();
  GCQ_TRY(timed_begin(ctx));
  {
    // the weighted sum keeps X unconjugated (the conjugation is applied per slice)
    std::vector<int> zero(L, 0);
    GCQ_TRY(upload(ctx->scratchD, zero, st));
    if (precision == GCQ_C128)
      hipLaunchKernelGGL((perm_in3<double, T>), dim3(g), dim3(256), 0, st, (const cpx<double>*)X,
                         Xp, perm, ctx->scratchD.as<int>(), n, L);
    else
      hipLaunchKernelGGL((perm_in3<float, T>), dim3(g), dim3(256), 0, st, (const cpx<float>*)X, Xp,
                         perm, ctx->scratchD.as<int>(), n, L);
    hipLaunchKernelGGL(zero3<T>, dim3(64), dim3(256), 0, st, Yp, int64_t(n));
    auto wsum = [&](auto kern, int nt) {
      hipLaunchKernelGGL(kern, dim3(wgrid), dim3(nt), 0, st, ctx->d_blk.as<int>(), F.d_mvorder.as<int>(), nmv,
                         F.d_bterm.as<int>(), F.d_trank.as<int>(), F.d_toff.as<int64_t>(), F.d_tvoff.as<int64_t>(),
                         F.d_tfoff.as<int64_t>(), F.slices.as<cpx<T>>(), d_colpos, d_conj, L, n, Xp, Yp);
    };
    // Many narrow blocks at few frequencies: a wave and two terms at a time, where
    // four waves and their barriers find too little work in a block.  The line, by
    // the mean side of the near blocks (a leaf's width) times the frequencies and by
    // the blocks, in us, one wave / four waves: 18000 triangles in leaves of 18 at 6
    // frequencies 882 / 1497, 8133 in leaves of 32 at 8 1352 / 1643, 10972 in leaves
    // of 21 at 10 1710 / 1735; 6661 in leaves of 26 at 14 1445 / 1011, 720 (few
    // blocks) in leaves of 22 at 6 86 / 73.
    const double side = std::sqrt(double(ctx->near_total) / std::max<size_t>(ctx->near_ids.size(), 1));
    if (nmv >= 4 * ctx->cus && side * L <= 260.0)
      wsum(wsum_kernel<T, 64, 2, 64, 32>, 64);
    else
      wsum(wsum_kernel<T, 256, 8, 128, 64>, 256);
    if (precision == GCQ_C128)
      hipLaunchKernelGGL((perm_out3<T, double>), dim3(64), dim3(256), 0, st, Yp, (cpx<double>*)Y,
                         perm, ctx->scratchD.as<int>(), n, 1);
    else
      hipLaunchKernelGGL((perm_out3<T, float>), dim3(64), dim3(256), 0, st, Yp, (cpx<float>*)Y,
                         perm, ctx->scratchD.as<int>(), n, 1);
  }
  GCQ_HIP(hipGetLastError());
  timed_end(ctx, "matvec_wsum");
  return GCQ_OK;
}

// the per-frequency product's buffers and tables, ahead of a capture
int prepare_perfreq(gcq_context* ctx, int precision) {
  if (ctx->F.precision != storage_precision(precision))
    return fail(GCQ_ERR_ARG, "precision differs from the one the 3D-ACA was built in");
  const int n = ctx->n, L = ctx->L;
  if (precision == GCQ_C64_SPLIT_BF16) {
    GCQ_TRY(bf16_setup(ctx));
    return product_setup(ctx, bf16_buffer_bytes(ctx));
  }
  return product_setup(ctx, size_t(2) * n * L * (precision == GCQ_C128 ? 16 : 8));
}

// the per-frequency product's kernels on stream s (no allocation, no host
// transfer: capturable after prepare_perfreq)
void enqueue_perfreq_any(gcq_context* ctx, hipStream_t s, int precision, const void* X, void* Y,
                         const int* tile_mask) {
  if (precision == GCQ_C64_SPLIT_BF16)
    enqueue_perfreq_bf16(ctx, s, X, Y, tile_mask);
  else if (precision == GCQ_C128)
    enqueue_perfreq<double>(ctx, s, precision, X, Y);
  else
    enqueue_perfreq<float>(ctx, s, precision, X, Y);
}

int run_compressed(gcq_context* ctx, int mode, int precision, const void* X, void* Y) {
  if (ctx->F.precision != storage_precision(precision))
    return fail(GCQ_ERR_ARG, "precision differs from the one the 3D-ACA was built in");
  if (precision == GCQ_C64_SPLIT_BF16 && mode != GCQ_PER_FREQUENCY)
    return fail(GCQ_ERR_UNSUPPORTED, "split-bf16 products are per frequency only");
  return precision == GCQ_C128 ? compressed_impl<double>(ctx, mode, precision, X, Y)
                               : compressed_impl<float>(ctx, mode, precision, X, Y);
}

}  // namespace gcq
