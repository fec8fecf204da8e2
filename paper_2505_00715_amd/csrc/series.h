// One panel pair at many frequencies.
//
// A pair's quadrature sum at frequency sigma = s / c is sum_q f_q exp(-sigma r_q)
// with weights f_q and distances r_q that do not depend on the frequency.  With
// r_q = r0 + h t_q, |t_q| <= 1, and z = -sigma h,
//   sum_q f_q exp(-sigma r_q) = exp(-sigma r0) sum_m z^m c_m,   c_m = sum_q f_q t_q^m / m!,
// so that after the moments c_m one exponential and one polynomial of degree D
// replace an exponential per quadrature point.  The double layer's factor
// 1 + sigma r_q adds the polynomial's derivative:
//   exp(-sigma r0) [(1 + sigma r0) P(z) - z P'(z)].
// All of it in float64.  The truncated part is below |z|^(D + 1) / (D + 1)! and
// rounding grows like exp(|z|), so that each result type has its largest |z|
// (SeriesLimit): 1 for double results, 3.5 for float ones, whose own rounding is
// far above the series' error.  Beyond it the near rule's points are put into
// several bins of smaller h, and the far rule's are summed one by one.  Double
// far-tier entries are always summed one by one: one exponential's rounding in
// place of the mean of seven raised their error by up to a tenth (2-norm against
// 80-bit values); the near tier's 112 points in bins lower theirs.
#pragma once
#include "device_common.h"

namespace gcq {

// 1 / m!
__device__ constexpr double SERIES_IF[24] = {
    1.0, 1.0, 1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720, 1.0 / 5040, 1.0 / 40320, 1.0 / 362880,
    1.0 / 3628800, 1.0 / 39916800, 1.0 / 479001600, 1.0 / 6227020800.0, 1.0 / 87178291200.0,
    1.0 / 1307674368000.0, 1.0 / 20922789888000.0, 1.0 / 355687428096000.0, 1.0 / 6402373705728000.0,
    1.0 / 121645100408832000.0, 1.0 / 2432902008176640000.0, 1.0 / 51090942171709440000.0,
    1.0 / 1124000727777607680000.0, 1.0 / 25852016738884976640000.0};

// the largest degree and the largest |z| it serves: the truncated part stays
// below 1e-9 (float results) and 5e-17 (double results) of the leading term; the
// far tier takes smaller degrees where its |z| allows them
template <typename T>
struct SeriesLimit;
template <>
struct SeriesLimit<float> {
  static constexpr int D0 = 8, D1 = 14, D2 = 22;
  static constexpr double Z0 = 0.41, Z1 = 1.6, Z2 = 3.5;
};
template <>
struct SeriesLimit<double> {
  static constexpr int D2 = 18;
  static constexpr double Z2 = 1.0;
};
// fewest frequencies that pay for a far pair's moments
constexpr int SERIES_MIN_F = 4;
constexpr int SERIES_BINS = 12;   // most bins of a near pair

// exp(-sigma r) = er (ec - i es) for double results: the products sigma r carry
// their rounding errors along (fma residuals)
__device__ __forceinline__ void cexp_pair(double r, double2 s, double& re, double& im) {
  const double pr = s.x * r, er = fma(s.x, r, -pr);
  const double pi = s.y * r, ei = fma(s.y, r, -pi);
  double sn, cs;
  sincos(pi, &sn, &cs);
  double e = exp(-pr);
  e = fma(-e, er, e);
  re = e * fma(-sn, ei, cs);
  im = -e * fma(cs, ei, sn);
}

// the same for float results: arguments reduced in double, then float
// polynomials (sine and cosine by their power series on [-pi/4, pi/4], the last
// terms kept below 3e-9) and the hardware exp2
__device__ __forceinline__ void cexp_float(double r, double2 s, double& re, double& im) {
  const double te = fmax(-s.x * r * 1.4426950408889634074, -1000.0);
  const double ne = rint(te);
  const float e = ldexpf(__builtin_amdgcn_exp2f(float(te - ne)), int(ne));
  const double tp = s.y * r * 0.15915494309189533577;   // revolutions
  const float fp = float(tp - rint(tp));
  const float q = rintf(4.f * fp);
  const float x = 6.283185307179586f * (fp - 0.25f * q), x2 = x * x;
  float sn = 1.f / 362880;
  sn = fmaf(sn, x2, -1.f / 5040);
  sn = fmaf(sn, x2, 1.f / 120);
  sn = fmaf(sn, x2, -1.f / 6);
  sn = fmaf(sn * x2, x, x);
  float cs = -1.f / 3628800;
  cs = fmaf(cs, x2, 1.f / 40320);
  cs = fmaf(cs, x2, -1.f / 720);
  cs = fmaf(cs, x2, 1.f / 24);
  cs = fmaf(cs, x2, -0.5f);
  cs = fmaf(cs, x2, 1.f);
  const int k = int(q) & 3;
  const float a = (k & 1) ? sn : cs, b = (k & 1) ? cs : sn;
  re = double(e * ((k == 1 || k == 2) ? -a : a));
  im = double(-e * ((k & 2) ? -b : b));
}

template <typename T>
__device__ __forceinline__ void cexp_to(double r, double2 s, double& re, double& im) {
  if constexpr (sizeof(T) == 4)
    cexp_float(r, s, re, im);
  else
    cexp_pair(r, s, re, im);
}

// exp(-sigma r0) times the polynomial's value (and derivative), as above
template <typename T, bool DLP, int D, typename Coef>
__device__ __forceinline__ void series_eval(const Coef& c, double r0, double h, double2 s, double& re, double& im) {
  const double zr = -s.x * h, zi = -s.y * h;
  double pr = c(D), pi = 0.0, qr = 0.0, qi = 0.0;
#pragma unroll
  for (int m = D - 1; m >= 0; --m) {
    if constexpr (DLP) {
      const double t = fma(qr, zr, fma(-qi, zi, pr));
      qi = fma(qr, zi, fma(qi, zr, pi));
      qr = t;
    }
    const double t = fma(pr, zr, fma(-pi, zi, c(m)));
    pi = fma(pr, zi, pi * zr);
    pr = t;
  }
  if constexpr (DLP) {
    const double ar = fma(s.x, r0, 1.0), ai = s.y * r0;
    const double t = ar * pr - ai * pi - (zr * qr - zi * qi);
    pi = ar * pi + ai * pr - (zr * qi + zi * qr);
    pr = t;
  }
  double er, ei;
  cexp_to<T>(r0, s, er, ei);
  re = pr * er - pi * ei;
  im = pr * ei + pi * er;
}

// one point's share f exp(-sigma r), times 1 + sigma r for the double layer
template <typename T, bool DLP>
__device__ __forceinline__ void point_add(double r, double f, double2 s, double& re, double& im) {
  double er, ei;
  if constexpr (sizeof(T) == 4) {
    cexp_float(r, s, er, ei);
  } else {
    double sn, cs;
    sincos(s.y * r, &sn, &cs);
    er = exp(-s.x * r);
    ei = -er * sn;
    er *= cs;
  }
  if constexpr (DLP) {
    const double ar = fma(s.x, r, 1.0), ai = s.y * r;
    const double t = ar * er - ai * ei;
    ei = ar * ei + ai * er;
    er = t;
  }
  re = fma(f, er, re);
  im = fma(f, ei, im);
}

// LDS of the far tier's distances and weights: [14][threads] (float results)
constexpr int FAR_THREADS = 256;
template <typename T>
constexpr int far_pts() { return sizeof(T) == 4 ? 2 * NQ_FAR * FAR_THREADS : 1; }

template <bool DLP, int D, typename Store>
__device__ __forceinline__ void far_series(const double* __restrict__ pts, double r0, double h, double hmax, bool ok,
                                           const double2* __restrict__ sig, int k0, int nf, int kstep,
                                           const Store& store) {
  double c[D + 1];
  {
    const double ih = h > 0.0 ? 1.0 / h : 0.0;
#pragma unroll
    for (int m = 0; m <= D; ++m) c[m] = 0.0;
#pragma unroll 1
    for (int q = 0; q < NQ_FAR; ++q) {
      const double t = (pts[q * FAR_THREADS] - r0) * ih;
      double pw = pts[(NQ_FAR + q) * FAR_THREADS];
#pragma unroll
      for (int m = 0; m <= D; ++m) {
        c[m] += pw;
        pw *= t;
      }
    }
#pragma unroll
    for (int m = 2; m <= D; ++m) c[m] *= SERIES_IF[m];
  }
  constexpr double Z = SeriesLimit<float>::Z2;
  const double lim = hmax > 0.0 ? Z * Z / (hmax * hmax) : 1e300;
  for (int k = k0; k < nf; k += kstep) {
    const double2 s = sig[k];
    double re = 0.0, im = 0.0;
    if (s.x * s.x + s.y * s.y <= lim) {
      series_eval<float, DLP, D>([&](int m) { return c[m]; }, r0, h, s, re, im);
    } else {
#pragma unroll 1
      for (int q = 0; q < NQ_FAR; ++q)
        point_add<float, DLP>(pts[q * FAR_THREADS], pts[(NQ_FAR + q) * FAR_THREADS], s, re, im);
    }
    if (ok) store(k, cpx<float>{float(re), float(im)});
  }
}

// far-tier entry (pi, pj) at the frequencies k0, k0 + kstep, .. below nf, one pair
// per thread of a workgroup of FAR_THREADS; every lane of the wave calls (ok: the
// lane holds a pair).  smax = max |sigma|.  Float results: the degree and the
// test |z| <= limit go by the wave's largest h, so that they are uniform; pts
// holds the thread's distances and weights in LDS, so that neither the moments
// nor the point-by-point sum unroll over them (91 registers instead of 147).
// Double results keep them in registers, unrolled (0.70 ms; from LDS 0.81 ms on the
// 1620-triangle sphere's near blocks at 16 frequencies).  store(k, value) per
// frequency.
template <typename T, bool DLP, typename Store>
__device__ __forceinline__ void far_pair(const Tab& tab, int pi, int pj, bool ok, const double2* __restrict__ sig,
                                         int k0, int nf, int kstep, double smax, double* pts, const Store& store) {
  const int n = tab.n;
  const double xi = tab.cen[pi], yi = tab.cen[n + pi], zi = tab.cen[2 * n + pi];
  double nrm[3] = {0.0, 0.0, 0.0};
  if constexpr (DLP) panel_normal(tab, pj, nrm);
  double r[NQ_FAR], f[NQ_FAR];
#pragma unroll
  for (int a = 0; a < NQ_FAR; ++a) {
    const double dx = xi - tab.q64[a * n + pj], dy = yi - tab.q64[(7 + a) * n + pj];
    const double dz = zi - tab.q64[(14 + a) * n + pj];
    const double r2 = dx * dx + dy * dy + dz * dz;
    r[a] = sqrt(r2);
    f[a] = tab.q64[(21 + a) * n + pj];
    if constexpr (DLP)
      f[a] *= (dx * nrm[0] + dy * nrm[1] + dz * nrm[2]) / (r2 * r[a]);
    else if constexpr (sizeof(T) == 4)
      f[a] /= r[a];
  }
  if constexpr (sizeof(T) == 8) {
    if (!ok) return;
    for (int k = k0; k < nf; k += kstep) {
      const double2 s = sig[k];
      double re = 0.0, im = 0.0;
#pragma unroll
      for (int a = 0; a < NQ_FAR; ++a) {
        const cpx<double> g = DLP ? dlp_radial(r[a], s.x, s.y) : green(r[a], s.x, s.y);
        re += f[a] * g.re;
        im += f[a] * g.im;
      }
      store(k, cpx<double>{re, im});
    }
  } else {
    double lo = r[0], hi = r[0];
#pragma unroll
    for (int a = 0; a < NQ_FAR; ++a) {
      lo = fmin(lo, r[a]);
      hi = fmax(hi, r[a]);
      pts[a * FAR_THREADS] = r[a];
      pts[(NQ_FAR + a) * FAR_THREADS] = f[a];
    }
    const double r0 = 0.5 * (lo + hi), h = 0.5 * (hi - lo);
    const double hmax = unid(wave_max(ok ? h : 0.0)), zw = smax * hmax;
    using SL = SeriesLimit<float>;
    if (zw <= SL::Z0)
      far_series<DLP, SL::D0>(pts, r0, h, hmax, ok, sig, k0, nf, kstep, store);
    else if (zw <= SL::Z1)
      far_series<DLP, SL::D1>(pts, r0, h, hmax, ok, sig, k0, nf, kstep, store);
    else
      far_series<DLP, SL::D2>(pts, r0, h, hmax, ok, sig, k0, nf, kstep, store);
  }
}

// Self or near-tier entry (pi, pj) at nf frequencies by one wave (pi, pj
// wave-uniform), in float64.  Near: 112 points, two per lane, in up to
// SERIES_BINS bins of equal width in r; the moments are wave sums, kept in
// `lds` (SERIES_LDS doubles of the wave's own); then a lane per frequency.  The
// self panel's angles (lanes 0..47) enter the same way: with R the distance to
// the edge, sum w R (1 - exp(-sigma R)) / (sigma R) = sum_m z^m / (m + 1)! sum w R t^m,
// t = R / h, h = max R.  Few frequencies, or more bins than fit: point by
// point, a point per lane and a wave sum per frequency.
constexpr int SERIES_LDS = SERIES_BINS * (SeriesLimit<float>::D2 + 1);
template <typename T, bool DLP, typename Store>
__device__ __forceinline__ void near_pair(const Tab& tab, int pi, int pj, const double2* __restrict__ sig, int nf,
                                          double smax, double* lds, const Store& store) {
  constexpr int D = SeriesLimit<T>::D2;
  const int n = tab.n, lane = threadIdx.x & (WAVE - 1);
  const bool self = pi == pj;
  if (DLP && self) {   // the centroid lies in its flat panel's plane
    for (int k = lane; k < nf; k += WAVE) store(k, cpx<T>{T(0), T(0)});
    return;
  }
  const double xi = tab.cen[pi], yi = tab.cen[n + pi], zi = tab.cen[2 * n + pi];
  double r[2] = {0.0, 0.0}, f[2] = {0.0, 0.0};
  bool in[2] = {false, false};
  if (self) {
    if (lane < 3 * NGL) {
      const int e = lane / NGL, g = lane % NGL, e1 = (e + 1) % 3;
      const double px = tab.vert[3 * e * n + pj] - xi, py = tab.vert[(3 * e + 1) * n + pj] - yi,
                   pz = tab.vert[(3 * e + 2) * n + pj] - zi;
      const double qx = tab.vert[3 * e1 * n + pj] - xi, qy = tab.vert[(3 * e1 + 1) * n + pj] - yi,
                   qz = tab.vert[(3 * e1 + 2) * n + pj] - zi;
      double ex = qx - px, ey = qy - py, ez = qz - pz;
      const double el = sqrt(ex * ex + ey * ey + ez * ez);
      ex /= el; ey /= el; ez /= el;
      const double tp = px * ex + py * ey + pz * ez, tq = qx * ex + qy * ey + qz * ez;
      const double fx = px - tp * ex, fy = py - tp * ey, fz = pz - tp * ez;
      const double d = sqrt(fx * fx + fy * fy + fz * fz);
      const double ta = atan2(tp, d), span = atan2(tq, d) - ta;
      r[0] = d / cos(ta + span * tab.K->gl_x[g]);
      f[0] = span * tab.K->gl_w[g] * r[0] * INV4PI;
      in[0] = true;
    }
  } else {
    double v[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) v[c] = tab.vert[c * n + pj];
    double nrm[3] = {0.0, 0.0, 0.0};
    if constexpr (DLP) panel_normal(tab, pj, nrm);
    const double wa = tab.area[pj] * INV4PI;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int a = lane + q * WAVE;
      in[q] = a < NQ_NEAR;
      if (!in[q]) continue;
      const double b0 = tab.K->nb[a][0], b1 = tab.K->nb[a][1], b2 = tab.K->nb[a][2];
      const double dx = xi - (b0 * v[0] + b1 * v[3] + b2 * v[6]);
      const double dy = yi - (b0 * v[1] + b1 * v[4] + b2 * v[7]);
      const double dz = zi - (b0 * v[2] + b1 * v[5] + b2 * v[8]);
      const double r2 = dx * dx + dy * dy + dz * dz;
      r[q] = sqrt(r2);
      f[q] = tab.K->nw[a] * wa / r[q];
      if constexpr (DLP) f[q] *= (dx * nrm[0] + dy * nrm[1] + dz * nrm[2]) / r2;
    }
  }
  const double hi = unid(wave_max(fmax(in[0] ? r[0] : 0.0, in[1] ? r[1] : 0.0)));
  const double lo = self ? -hi : -unid(wave_max(fmax(in[0] ? -r[0] : -1e300, in[1] ? -r[1] : -1e300)));
  const double half = 0.5 * (hi - lo);   // self: bins about r = 0, half = max R
  const double want = smax * half / SeriesLimit<T>::Z2;
  const int nb = want > 1.0 ? int(fmin(ceil(want), 1e6)) : 1;
  if (nf < 4 * nb || nb > (self ? 1 : SERIES_BINS)) {
    for (int k = 0; k < nf; ++k) {
      const double2 s = sig[k];
      double re = 0.0, im = 0.0;
      if (self) {
        if (in[0]) {
          const cpx<double> p = phi_c(s.x * r[0], s.y * r[0]);
          re = f[0] * p.re;
          im = f[0] * p.im;
        }
      } else {
#pragma unroll
        for (int q = 0; q < 2; ++q)
          if (in[q]) point_add<double, DLP>(r[q], f[q], s, re, im);
      }
      re = wave_sum(re);
      im = wave_sum(im);
      if (lane == 0) store(k, cpx<T>{T(re), T(im)});
    }
    return;
  }
  const double h = half / nb, ih = h > 0.0 ? 1.0 / h : 0.0;
  for (int b = 0; b < nb; ++b) {
    const double r0 = self ? 0.0 : lo + (2 * b + 1) * h;
    double t[2], pw[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const bool mine = in[q] && (self || min(int((r[q] - lo) * 0.5 * ih), nb - 1) == b);
      t[q] = (r[q] - r0) * ih;
      pw[q] = mine ? f[q] : 0.0;
      if (!mine) t[q] = 0.0;
    }
#pragma unroll 4
    for (int m = 0; m <= D; ++m) {
      const double s = wave_sum(pw[0] + pw[1]);
      pw[0] *= t[0];
      pw[1] *= t[1];
      if (lane == 0) lds[b * (D + 1) + m] = s * (self ? SERIES_IF[m + 1] : SERIES_IF[m]);
    }
  }
  __threadfence_block();
  __builtin_amdgcn_wave_barrier();
  for (int k = lane; k < nf; k += WAVE) {
    const double2 s = sig[k];
    double re = 0.0, im = 0.0;
    if (self) {
      const double zr = -s.x * h, zi = -s.y * h;
      re = lds[D];
#pragma unroll
      for (int m = D - 1; m >= 0; --m) {
        const double x = fma(re, zr, fma(-im, zi, lds[m]));
        im = fma(re, zi, im * zr);
        re = x;
      }
    } else {
      for (int b = 0; b < nb; ++b) {
        double vr, vi;
        series_eval<double, DLP, D>([&](int m) { return lds[b * (D + 1) + m]; }, lo + (2 * b + 1) * h, h, s, vr, vi);
        re += vr;
        im += vi;
      }
    }
    store(k, cpx<T>{T(re), T(im)});
  }
  __threadfence_block();
  __builtin_amdgcn_wave_barrier();   // the coefficients are free for the wave's next pair
}

}  // namespace gcq
