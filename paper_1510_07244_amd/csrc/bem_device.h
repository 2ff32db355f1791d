// Device helpers shared by the kernels (gfx950, wave64): reciprocal square
// root, sine/cosine, accumulators, pair classification, the Sauter-Schwab
// relabelling and the wave-cooperative singular-pair quadrature.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "bem_internal.h"

namespace bem {
namespace dev {

constexpr double kInv4Pi = 0.0795774715459476678844418816863;  // 1 / (4 pi)
constexpr int kThreads = 256;
constexpr int kWave = 64;

// 1/sqrt(a) for a > 0: hardware estimate (relative error below 6e-8) and one
// Newton step y (3 - a y^2) / 2, which leaves a relative error near 1e-15.
__device__ __forceinline__ double rsqrt_newton(double a) {
  const double y = __builtin_amdgcn_rsq(a);
  const double t = a * y;
  const double e = fma(-t, y, 1.0);
  return fma(0.5 * y, e, y);
}

// sin and cos of x: Cody-Waite reduction x = k pi + r, |r| <= pi/2, with pi
// split into three parts (the first two with 33 significant bits so that
// k * part is exact for |k| < 2^20), then sin r = r + r^3 P(r^2) and
// cos r = 1 - r^2 / 2 + r^4 Q(r^2), P of degree 7 minimising the error
// relative to sin r and Q of degree 6 minimising the absolute error of cos r
// on [-pi/2, pi/2] (Remez exchange on the Taylor tail, computed by
// sincos_minimax.py beside this file: below 5.4e-18 relative and 1.4e-17
// absolute with the coefficients rounded to double); odd k negates both,
// by the sign bit.  Reducing by pi rather than pi/2 costs two more
// polynomial terms and saves the quadrant's exchange of sine and cosine.
constexpr double kOneOverPi = 0.31830988618379067154;
constexpr double kPia = 3.1415926534682512;      // 0x1.921fb544p+1
constexpr double kPib = 1.2154201012607932e-10;  // 0x1.0b4611a6p-33
constexpr double kPic = 4.044532497591901e-21;   // 0x1.3198a2e037073p-68

// x with its sign flipped when bit 31 of sgn is set
__device__ __forceinline__ double flip_sign(double x, int sgn) {
  return __hiloint2double(__double2hiint(x) ^ sgn, __double2loint(x));
}

__device__ __forceinline__ void sincos_cw(double x, double *s, double *c) {
  const double k = __builtin_rint(x * kOneOverPi);
  double r = fma(-k, kPia, x);
  r = fma(-k, kPib, r);
  r = fma(-k, kPic, r);
  const double r2 = r * r;
  double ps = 0x1.8829a2ffb2991p-49;  // P, highest degree first
  ps = fma(ps, r2, -0x1.ae431d98dda7bp-41);
  ps = fma(ps, r2, 0x1.6123cb29045c6p-33);
  ps = fma(ps, r2, -0x1.ae6454cb574e2p-26);
  ps = fma(ps, r2, 0x1.71de3a5287c76p-19);
  ps = fma(ps, r2, -0x1.a01a01a0148bcp-13);
  ps = fma(ps, r2, 0x1.11111111110c1p-7);
  ps = fma(ps, r2, -0x1.5555555555555p-3);
  const double sr = fma(r * r2, ps, r);
  double pc = 0x1.9fc8d3c9114a6p-45;  // Q, highest degree first
  pc = fma(pc, r2, -0x1.93573fa1f69b4p-37);
  pc = fma(pc, r2, 0x1.1eecfaec8e87dp-29);
  pc = fma(pc, r2, -0x1.27e4f9f33e2edp-22);
  pc = fma(pc, r2, 0x1.a01a019ba7403p-16);
  pc = fma(pc, r2, -0x1.6c16c16c10218p-10);
  pc = fma(pc, r2, 0x1.55555555554ddp-5);
  pc = fma(pc, r2, -0.5);
  const double cr = fma(r2, pc, 1.0);
  const int sgn = static_cast<int>((static_cast<unsigned>(static_cast<int>(k)) & 1u) << 31);
  *s = flip_sign(sr, sgn);
  *c = flip_sign(cr, sgn);
}

// FP32 sine and cosine for the mixed-precision path: the same reduction by
// pi, truncated to 12 + 12 + 24 significant bits (k * part exact for
// |k| < 2^12), minimax P and Q of degree 3 from the same construction (errors
// below 9.7e-9 relative and 5.8e-9 absolute with the coefficients rounded to
// float).
__device__ __forceinline__ void sincos_cw_f32(float x, float *s, float *c) {
  const float k = __builtin_rintf(x * 0.31830988f);
  float r = fmaf(-k, 3.140625f, x);               // 0x1.92p+1
  r = fmaf(-k, 9.67502593994140625e-4f, r);       // 0x1.fb4p-11
  r = fmaf(-k, 1.5099579e-7f, r);                 // 0x1.4442dp-23
  const float r2 = r * r;
  float ps = 0x1.5dbdf0p-19f;
  ps = fmaf(ps, r2, -0x1.9f6ffep-13f);
  ps = fmaf(ps, r2, 0x1.110ed4p-7f);
  ps = fmaf(ps, r2, -0x1.55554cp-3f);
  const float sr = fmaf(r * r2, ps, r);
  float pc = -0x1.194102p-22f;
  pc = fmaf(pc, r2, 0x1.9f8f5ap-16f);
  pc = fmaf(pc, r2, -0x1.6c149cp-10f);
  pc = fmaf(pc, r2, 0x1.555550p-5f);
  pc = fmaf(pc, r2, -0.5f);
  const float cr = fmaf(r2, pc, 1.0f);
  const int sgn = static_cast<int>((static_cast<unsigned>(static_cast<int>(k)) & 1u) << 31);
  *s = __int_as_float(__float_as_int(sr) ^ sgn);
  *c = __int_as_float(__float_as_int(cr) ^ sgn);
}

// Sine and cosine of a phase |x| <= 3/4 relative to a reference distance, no
// reduction: sin x = x + x^3 P(x^2), cos x = 1 - x^2 / 2 + x^4 Q(x^2), P and Q
// from the same construction on [0, 9/16] (below 3.3e-18 relative and 4.1e-17
// absolute; FP32 6.9e-9 and 5.0e-10): 14 instructions (FP32 9) where the
// reduction by pi and its polynomials take 28 (20).
constexpr double kShortPhase = 0.75;
__device__ __forceinline__ void short_phase(double x, double *s, double *c) {
  const double r2 = x * x;
  double ps = 0x1.5de07ede42fd2p-33;
  ps = fma(ps, r2, -0x1.ae5f5cd1da528p-26);
  ps = fma(ps, r2, 0x1.71de36994cee9p-19);
  ps = fma(ps, r2, -0x1.a01a019d434f0p-13);
  ps = fma(ps, r2, 0x1.111111111012cp-7);
  ps = fma(ps, r2, -0x1.555555555554ep-3);
  *s = fma(x * r2, ps, x);
  double pc = 0x1.1c0e6d71989eep-29;
  pc = fma(pc, r2, -0x1.27e0f9998bd9dp-22);
  pc = fma(pc, r2, 0x1.a019fc581f756p-16);
  pc = fma(pc, r2, -0x1.6c16c168dbc4bp-10);
  pc = fma(pc, r2, 0x1.5555555553e74p-5);
  pc = fma(pc, r2, -0.5);
  *c = fma(r2, pc, 1.0);
}
__device__ __forceinline__ void short_phase_f32(float x, float *s, float *c) {
  const float r2 = x * x;
  float ps = -0x1.99dddcp-13f;
  ps = fmaf(ps, r2, 0x1.1108e4p-7f);
  ps = fmaf(ps, r2, -0x1.55554ap-3f);
  *s = fmaf(x * r2, ps, x);
  float pc = 0x1.9a8ae2p-16f;
  pc = fmaf(pc, r2, -0x1.6c0e42p-10f);
  pc = fmaf(pc, r2, 0x1.55554ep-5f);
  pc = fmaf(pc, r2, -0.5f);
  *c = fmaf(r2, pc, 1.0f);
}

template <int KERNEL>
struct Acc;
template <>
struct Acc<BEM_LAPLACE> {
  double re = 0.0;
};
template <>
struct Acc<BEM_HELMHOLTZ> {
  double re = 0.0, im = 0.0;
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = kWave / 2; o >= 1; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

template <int KERNEL>
__device__ __forceinline__ void store(void *out, int64_t k, const Acc<KERNEL> &v,
                                      unsigned *flags) {
  if constexpr (KERNEL == BEM_LAPLACE) {
    if (!isfinite(v.re)) atomicOr(flags, FLAG_NONFINITE);
    static_cast<double *>(out)[k] = v.re;
  } else {
    if (!isfinite(v.re) || !isfinite(v.im)) atomicOr(flags, FLAG_NONFINITE);
    static_cast<double2 *>(out)[k] = make_double2(v.re, v.im);
  }
}

// Store for the plain (double / double2) or mixed (float / float2) output.
template <int KERNEL, bool MIXED>
__device__ __forceinline__ void store_as(void *out, int64_t k, const Acc<KERNEL> &v,
                                         unsigned *flags) {
  if constexpr (!MIXED) {
    store<KERNEL>(out, k, v, flags);
  } else if constexpr (KERNEL == BEM_LAPLACE) {
    const float r = static_cast<float>(v.re);
    if (!isfinite(r)) atomicOr(flags, FLAG_NONFINITE);
    static_cast<float *>(out)[k] = r;
  } else {
    const float r = static_cast<float>(v.re), i = static_cast<float>(v.im);
    if (!isfinite(r) || !isfinite(i)) atomicOr(flags, FLAG_NONFINITE);
    static_cast<float2 *>(out)[k] = make_float2(r, i);
  }
}

typedef const double __attribute__((address_space(4))) *uniform_ptr;

constexpr int kSS = 2;  // layer value: both layers

// Sums over the column points y_b of one x-point (lane's own), without the
// x-point's weight: single layer s, double layer d, and with P1 the same
// kernel values times the column triangle's barycentric coordinates.
struct RowSum {
  double sr[3], si[3], dr[3], di[3];
};

// Orthonormal axes of a triangle's plane: e1 = l u and e2 = a u + b w up to
// rounding of their own size, n = u x w.  The second axis is orthogonalised
// twice and the third taken from the first two, so that both edges have no
// component along n beyond that rounding however flat the triangle is.
struct TriFrame {
  double u[3], w[3], n[3], l, a, b;
};
__device__ __forceinline__ double dot3(const double *a, const double *b) {
  return fma(a[0], b[0], fma(a[1], b[1], a[2] * b[2]));
}
__device__ __forceinline__ TriFrame tri_frame(const double *e1, const double *e2) {
  // two Newton steps: an error of the axes' length is one of every distance
  auto inv_sqrt = [](double x) {
    const double y = rsqrt_newton(x), e = fma(-(x * y), y, 1.0);
    return fma(0.5 * y, e, y);
  };
  TriFrame f;
  const double il = inv_sqrt(dot3(e1, e1));
#pragma unroll
  for (int c = 0; c < 3; ++c) f.u[c] = e1[c] * il, f.w[c] = e2[c];
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const double k = dot3(f.w, f.u);
#pragma unroll
    for (int c = 0; c < 3; ++c) f.w[c] = fma(-k, f.u[c], f.w[c]);
  }
  double b2 = dot3(f.w, f.w);
  if (b2 == 0.0) {  // flat to the last bit (its area is rounding): the axis that u has least of
    const double x = fabs(f.u[0]), y = fabs(f.u[1]), z = fabs(f.u[2]);
    const int k = x <= y && x <= z ? 0 : y <= z ? 1 : 2;
    const double uk = k == 0 ? f.u[0] : k == 1 ? f.u[1] : f.u[2];
#pragma unroll
    for (int c = 0; c < 3; ++c) f.w[c] = fma(-uk, f.u[c], c == k ? 1.0 : 0.0);
    b2 = dot3(f.w, f.w);
  }
  const double ib = inv_sqrt(b2);
#pragma unroll
  for (int c = 0; c < 3; ++c) f.w[c] *= ib;
  f.n[0] = fma(f.u[1], f.w[2], -f.u[2] * f.w[1]);
  f.n[1] = fma(f.u[2], f.w[0], -f.u[0] * f.w[2]);
  f.n[2] = fma(f.u[0], f.w[1], -f.u[1] * f.w[0]);
  f.l = dot3(e1, f.u);
  f.a = dot3(e2, f.u);
  f.b = dot3(e2, f.w);
  return f;
}

// One regular (disjoint) pair (i, j) in FP64 with its rule points formed from
// the geometry arrays, XC x-points at a time: the chunks sub, sub + G, ... of
// the rule's nq points (G lanes share a pair; each returns its part).
// Distances are sums of squared coordinate differences in axes of the column
// triangle's plane: an x-point's height above it is squared once, so a point
// pair takes two differences and two multiply-adds, and the height is
// <x - y, n_j> too.  Nothing cancels beyond the difference of the points
// itself (1/r to eps h / r at triangle size h): these are also the pairs that
// the mixed form leaves to FP64 because they are close.  A quadratic
// polynomial of the column's rule coordinates takes one operation less and loses
// eps (h / r)^2 (facing sheets 1e-4 h apart: 1e-8 where this and the plain
// difference lose 1e-13; NaN from 1e-8 h on) at the same speed: 1000 entries 10.4
// and 10.3 us, 300000 81.6 and 80.1, 440000 piecewise-linear pairs 120 and 124,
// mixed matrix step of 8192 triangles 2.01 ms both.  The rule is read by scalar
// loads.
// row(k, w, sums) is called for every x-point k with its weight (zero and a
// repeated point past the last one); with MIRROR *mr, *mi receive the double
// layer of (j, i), which needs the row's weights inside.
template <int KERNEL, int LAYER, bool MIRROR, bool P1, int XC, class F>
__device__ __forceinline__ void regular_rows(const double *g, int64_t L, const double *rule, int nq,
                                             double kappa, int i, int j, int sub, int G, F &&row,
                                             double *mr = nullptr, double *mi = nullptr) {
  constexpr int NB = P1 ? 3 : 1;
  constexpr bool S = LAYER != BEM_DLP, D = LAYER != BEM_SLP;
  const uniform_ptr R = (uniform_ptr)rule;
  double X0[3], e1i[3], e2i[3], e1j[3], e2j[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    X0[c] = g[(G_V0X + c) * L + i] - g[(G_V0X + c) * L + j];
    e1i[c] = g[(G_E1X + c) * L + i];
    e2i[c] = g[(G_E2X + c) * L + i];
    e1j[c] = g[(G_E1X + c) * L + j];
    e2j[c] = g[(G_E2X + c) * L + j];
  }
  const TriFrame f = tri_frame(e1j, e2j);
  // x - v0_j in the axes, linear in the row's rule coordinates
  const double p0 = dot3(X0, f.u), p1 = dot3(e1i, f.u), p2 = dot3(e2i, f.u);
  const double q0 = dot3(X0, f.w), q1 = dot3(e1i, f.w), q2 = dot3(e2i, f.w);
  const double h0 = dot3(X0, f.n), h1 = dot3(e1i, f.n), h2 = dot3(e2i, f.n);
  // <y - x, n_i> = m1 u + m2 v - m0
  double m0 = 0.0, m1 = 0.0, m2 = 0.0;
  if constexpr (MIRROR) {
    const TriFrame r = tri_frame(e1i, e2i);
    m0 = dot3(X0, r.n), m1 = dot3(e1j, r.n), m2 = dot3(e2j, r.n);
  }
  for (int a0 = sub * XC; a0 < nq; a0 += G * XC) {
    double p[XC], q[XC], h[XC], w[XC];
    RowSum acc[XC];
#pragma unroll
    for (int a = 0; a < XC; ++a) {
      const int k = min(a0 + a, nq - 1);
      // lanes of a pair take different x-points: per-lane loads
      const double s = rule[k], t = rule[nq + k];
      w[a] = a0 + a < nq ? rule[2 * nq + k] : 0.0;
      p[a] = fma(s, p1, fma(t, p2, p0));
      q[a] = fma(s, q1, fma(t, q2, q0));
      h[a] = fma(s, h1, fma(t, h2, h0));
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[a].sr[b] = acc[a].si[b] = acc[a].dr[b] = acc[a].di[b] = 0.0;
    }
    constexpr int U = XC == 1 ? 4 : 1;  // column points per step
    auto step = [&](int b0, int nu) {
      double u[U], v[U], wb[U], r2[U][XC], y[U][XC];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int b = U == 1 ? b0 : min(b0 + k, nq - 1);
        u[k] = R[b];
        v[k] = R[nq + b];
        wb[k] = k < nu ? R[2 * nq + b] : 0.0;
        const double yp = fma(u[k], f.l, v[k] * f.a), yq = v[k] * f.b;
#pragma unroll
        for (int a = 0; a < XC; ++a) {
          const double dp = p[a] - yp, dq = q[a] - yq;
          r2[k][a] = fma(dp, dp, fma(dq, dq, h[a] * h[a]));
        }
      }
#pragma unroll
      for (int k = 0; k < U; ++k)
#pragma unroll
        for (int a = 0; a < XC; ++a) y[k][a] = __builtin_amdgcn_rsq(r2[k][a]);
#pragma unroll
      for (int k = 0; k < U; ++k) {
        double tr = 0.0, ti = 0.0;
#pragma unroll
        for (int a = 0; a < XC; ++a) {
          const double z = fma(0.5 * y[k][a], fma(-(r2[k][a] * y[k][a]), y[k][a], 1.0), y[k][a]);
          double z3 = 0.0, cs = 1.0, sn = 0.0, fr = 1.0, fi = 0.0;
          if (D) z3 = z * z * z;
          if constexpr (KERNEL == BEM_HELMHOLTZ) {
            const double kr = kappa * r2[k][a] * z;
            sincos_cw(kr, &sn, &cs);
            if (D) fr = fma(kr, sn, cs), fi = fma(-kr, cs, sn);
          }
          auto add = [&](double f, double re, double im, double *ar, double *ai) {
            const double x = f * re;
            if constexpr (P1) {
              ar[0] += x;
              ar[1] = fma(u[k], x, ar[1]);
              ar[2] = fma(v[k], x, ar[2]);
            } else {
              ar[0] = fma(f, re, ar[0]);
            }
            if constexpr (KERNEL == BEM_HELMHOLTZ) {
              const double y = f * im;
              if constexpr (P1) {
                ai[0] += y;
                ai[1] = fma(u[k], y, ai[1]);
                ai[2] = fma(v[k], y, ai[2]);
              } else {
                ai[0] = fma(f, im, ai[0]);
              }
            }
          };
          if (S) add(wb[k] * z, cs, sn, acc[a].sr, acc[a].si);
          if (D) add(wb[k] * z3, fr, fi, acc[a].dr, acc[a].di);
          if (MIRROR) {
            const double x = w[a] * z3;
            tr = fma(x, fr, tr);
            if constexpr (KERNEL == BEM_HELMHOLTZ) ti = fma(x, fi, ti);
          }
        }
        if (MIRROR) {
          const double wm = wb[k] * fma(m1, u[k], fma(m2, v[k], -m0));
          *mr = fma(wm, tr, *mr);
          if constexpr (KERNEL == BEM_HELMHOLTZ) *mi = fma(wm, ti, *mi);
        }
      }
    };
    for (int b = 0; b < nq; b += U) step(b, nq - b);
#pragma unroll
    for (int a = 0; a < XC; ++a) {
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[a].dr[b] *= h[a], acc[a].di[b] *= h[a];
      row(min(a0 + a, nq - 1), w[a], acc[a]);
    }
  }
}

// sqrt(g_i g_j) / (4 pi) sum_a w_a sum_b w_b k(x_a, y_b) over the x-points of
// this lane (sub of G, see regular_rows); the lanes' parts add up to the entry.
template <int KERNEL, int LAYER, int XC = 4>
__device__ __forceinline__ Acc<KERNEL> regular_pair_fp64(const double *g, int64_t L,
                                                         const double *rule, int nq, double kappa,
                                                         int i, int j, int sub = 0, int G = 1) {
  double re = 0.0, im = 0.0;
  regular_rows<KERNEL, LAYER, false, false, XC>(g, L, rule, nq, kappa, i, j, sub, G,
                                                [&](int, double w, const RowSum &r) {
    re = fma(w, LAYER == BEM_SLP ? r.sr[0] : r.dr[0], re);
    if constexpr (KERNEL == BEM_HELMHOLTZ) im = fma(w, LAYER == BEM_SLP ? r.si[0] : r.di[0], im);
  });
  const double scale = g[G_SG * L + i] * g[G_SG * L + j] * kInv4Pi;
  Acc<KERNEL> v;
  v.re = re * scale;
  if constexpr (KERNEL == BEM_HELMHOLTZ) v.im = im * scale;
  return v;
}

// Both layers of (i, j) and the double layer of (j, i) in one pass.
template <int KERNEL>
__device__ __forceinline__ void regular_pair_both_fp64(const double *g, int64_t L, const double *rule,
                                                       int nq, double kappa, int i, int j,
                                                       Acc<KERNEL> *vs, Acc<KERNEL> *vd,
                                                       Acc<KERNEL> *vm) {
  double s[2] = {0, 0}, d[2] = {0, 0}, m[2] = {0, 0};
  regular_rows<KERNEL, kSS, true, false, 4>(g, L, rule, nq, kappa, i, j, 0, 1,
                                            [&](int, double w, const RowSum &r) {
    s[0] = fma(w, r.sr[0], s[0]);
    d[0] = fma(w, r.dr[0], d[0]);
    if constexpr (KERNEL == BEM_HELMHOLTZ) s[1] = fma(w, r.si[0], s[1]), d[1] = fma(w, r.di[0], d[1]);
  }, &m[0], &m[1]);
  const double f = g[G_SG * L + i] * g[G_SG * L + j] * kInv4Pi;
  vs->re = s[0] * f, vd->re = d[0] * f, vm->re = m[0] * f;
  if constexpr (KERNEL == BEM_HELMHOLTZ) vs->im = s[1] * f, vd->im = d[1] * f, vm->im = m[1] * f;
}

__device__ __forceinline__ int shared_vertex_count(int a0, int a1, int a2, int b0, int b1, int b2) {
  return (a0 == b0) + (a0 == b1) + (a0 == b2) + (a1 == b0) + (a1 == b1) + (a1 == b2) +
         (a2 == b0) + (a2 == b1) + (a2 == b2);
}

// rotate (t0, t1, t2) left by k in {0, 1, 2}, without indexing an array
__device__ __forceinline__ void rotate3(int t0, int t1, int t2, int k, int *o0, int *o1, int *o2) {
  *o0 = k == 0 ? t0 : (k == 1 ? t1 : t2);
  *o1 = k == 0 ? t1 : (k == 1 ? t2 : t0);
  *o2 = k == 0 ? t2 : (k == 1 ? t0 : t1);
}

// Relabelling of a singular pair (common vertices first):
//   identical: mesh order; edge: the common vertices (lo, hi) by global id,
//   then the third vertex; vertex: the common vertex, then the other two in
//   the mesh's cyclic order.
__device__ __forceinline__ void relabel(int i0, int i1, int i2, int j0, int j1, int j2, int cls,
                                        int li[3], int lj[3]) {
  if (cls == CLS_IDENTICAL) {
    li[0] = i0, li[1] = i1, li[2] = i2;
    lj[0] = j0, lj[1] = j1, lj[2] = j2;
    return;
  }
  const bool s0 = i0 == j0 || i0 == j1 || i0 == j2;
  const bool s1 = i1 == j0 || i1 == j1 || i1 == j2;
  const bool s2 = i2 == j0 || i2 == j1 || i2 == j2;
  if (cls == CLS_EDGE) {
    const int ca = s0 ? i0 : i1;            // first common vertex in i's order
    const int cb = s2 ? i2 : (s1 && s0 ? i1 : i2);
    const int lo = min(ca, cb), hi = max(ca, cb);
    const int ci = !s0 ? i0 : (!s1 ? i1 : i2);
    const bool r0 = j0 == lo || j0 == hi, r1 = j1 == lo || j1 == hi;
    const int cj = !r0 ? j0 : (!r1 ? j1 : j2);
    li[0] = lo, li[1] = hi, li[2] = ci;
    lj[0] = lo, lj[1] = hi, lj[2] = cj;
    return;
  }
  const int ka = s0 ? 0 : (s1 ? 1 : 2);
  const int a = ka == 0 ? i0 : (ka == 1 ? i1 : i2);
  const int kb = j0 == a ? 0 : (j1 == a ? 1 : 2);
  rotate3(i0, i1, i2, ka, &li[0], &li[1], &li[2]);
  rotate3(j0, j1, j2, kb, &lj[0], &lj[1], &lj[2]);
}

// ---------------------------------------------------------- Sauter-Schwab
// After relabelling, both affine maps start at a common vertex and the rule
// factors (singular_rule): x - y = p d(eta) with p a product of the rule's
// radial nodes and
//   d = g1 E1_i + g2 E2_i - g3 E1_j - g4 E2_j
// over 2 q^3 directions for a common vertex, 5 q^2 for a common edge (where
// E1_i = E1_j and g3 = 0) and 3 q for an identical pair (g3 = g4 = 0).  The
// Laplace kernels' radial sums are moments; the Helmholtz kernels' are power
// series in theta = kappa |d| whose coefficients hold the rule's own radial
// nodes (no other quadrature), taken up to theta = 2, where the terms left out
// are below 3e-17 of the sum and 6e-17 of its real part at every order (vertex
// pairs; 2e-18 the others); a larger theta sums the radial nodes.
struct PairGeo {
  double E1i[3], E2i[3], E1j[3], E2j[3], n[3];
  double scale;  // sqrt(g_i) sqrt(g_j) / (4 pi)
};

// Loads and relabels pair (i, j) of class cls; false (and the flag) if a
// vertex id is out of range.
__device__ __forceinline__ bool pair_geometry(const double *v, const int32_t *tri, int nv,
                                              const double *geo, int64_t ldg, int i, int j,
                                              int cls, unsigned *flags, PairGeo *g) {
  const int i0 = tri[3 * (int64_t)i], i1 = tri[3 * (int64_t)i + 1], i2 = tri[3 * (int64_t)i + 2];
  const int j0 = tri[3 * (int64_t)j], j1 = tri[3 * (int64_t)j + 1], j2 = tri[3 * (int64_t)j + 2];
  const bool ok = i0 >= 0 && i0 < nv && i1 >= 0 && i1 < nv && i2 >= 0 && i2 < nv && j0 >= 0 &&
                  j0 < nv && j1 >= 0 && j1 < nv && j2 >= 0 && j2 < nv;
  if (!ok) {
    atomicOr(flags, FLAG_EINVAL);
    return false;
  }
  int li[3], lj[3];
  relabel(i0, i1, i2, j0, j1, j2, cls, li, lj);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double pi0 = v[3 * (int64_t)li[0] + c], pi1 = v[3 * (int64_t)li[1] + c],
                 pi2 = v[3 * (int64_t)li[2] + c];
    const double pj0 = v[3 * (int64_t)lj[0] + c], pj1 = v[3 * (int64_t)lj[1] + c],
                 pj2 = v[3 * (int64_t)lj[2] + c];
    g->E1i[c] = pi1 - pi0;
    g->E2i[c] = pi2 - pi1;
    g->E1j[c] = pj1 - pj0;
    g->E2j[c] = pj2 - pj1;
  }
  g->n[0] = geo[G_NX * ldg + j];
  g->n[1] = geo[G_NY * ldg + j];
  g->n[2] = geo[G_NZ * ldg + j];
  g->scale = geo[G_SG * ldg + i] * geo[G_SG * ldg + j] * kInv4Pi;
  return true;
}

// Element k of a four-entry argument array by selects, not by an index: a
// kernel that copies its arguments into registers (the persistent form) would
// otherwise keep the whole copy in scratch memory.
template <class T>
__device__ __forceinline__ T pick4(const T (&v)[4], int k) {
  return k == 0 ? v[0] : k == 1 ? v[1] : k == 2 ? v[2] : v[3];
}

// Largest squared distance of a point of tau_i from one of tau_j: between two
// vertices (every direction d of the rule is such a difference).
__device__ __forceinline__ double pair_extent2(const PairGeo &g) {
  double m = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      double r2 = 0.0;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double x = a == 0 ? 0.0 : a == 1 ? g.E1i[c] : g.E1i[c] + g.E2i[c];
        const double y = b == 0 ? 0.0 : b == 1 ? g.E1j[c] : g.E1j[c] + g.E2j[c];
        r2 = fma(x - y, x - y, r2);
      }
      m = fmax(m, r2);
    }
  return m;
}

// Sums of a singular pair over directions: single layer, double layer of
// (i, j), and (with MIRROR) the double layer of (j, i) over the same
// directions (vertex pairs: the rule is symmetric).
struct SSSum {
  double sr = 0.0, si = 0.0, dr = 0.0, di = 0.0, mr = 0.0, mi = 0.0;
};

// Direction p of the table; VERTEX: four coefficients.
template <bool VERTEX, class P>
__device__ __forceinline__ void ss_direction(const PairGeo &g, P T, int n, int p, double d[3]) {
  const double g1 = T[p], g2 = T[n + p], g4 = T[3 * n + p];
  if constexpr (VERTEX) {
    const double g3 = T[2 * n + p];
#pragma unroll
    for (int c = 0; c < 3; ++c)
      d[c] = fma(g1, g.E1i[c], fma(g2, g.E2i[c], fma(-g3, g.E1j[c], -g4 * g.E2j[c])));
  } else {
#pragma unroll
    for (int c = 0; c < 3; ++c) d[c] = fma(g1, g.E1i[c], fma(g2, g.E2i[c], -g4 * g.E2j[c]));
  }
}

// Adds direction d with squared length r2, hardware estimate h of 1/|d| and
// weight w.  LAYER: BEM_SLP, BEM_DLP or kSS (both).  SER: Helmholtz by the
// power series, else over the radial nodes.  m: normal of tau_i (MIRROR).
template <int KERNEL, int LAYER, bool MIRROR, bool SER, class P>
__device__ __forceinline__ void ss_add(const PairGeo &g, const double d[3], double r2, double h,
                                       double w, P S, P R, int nr, double kappa, const double *m,
                                       SSSum *a) {
  // one Newton step: z = h + h (1 - r2 h^2) / 2 ~ 1 / |d|
  const double z = fma(0.5 * h, fma(-(r2 * h), h, 1.0), h);
  double wd = 0.0, wm = 0.0, z3 = 0.0;
  if constexpr (LAYER != BEM_SLP) {
    wd = w * fma(d[0], g.n[0], fma(d[1], g.n[1], d[2] * g.n[2]));
    if constexpr (MIRROR) wm = -w * fma(d[0], m[0], fma(d[1], m[1], d[2] * m[2]));
    z3 = z * z * z;
  }
  if constexpr (KERNEL == BEM_LAPLACE) {
    if constexpr (LAYER != BEM_DLP) a->sr = fma(w, z, a->sr);
    if constexpr (LAYER != BEM_SLP) a->dr = fma(wd, z3, a->dr);
    if constexpr (MIRROR) a->mr = fma(wm, z3, a->mr);
  } else if constexpr (SER) {
    // even and odd series in t = theta^2; the odd ones lack a factor theta
    // (single layer) resp. theta^3 (double layer: no linear term), put back
    // by ss_finish as kappa and kappa^3 with the powers of 1 / |d|
    const double t = kappa * kappa * r2;
    constexpr int N = kSeries;
    if constexpr (LAYER != BEM_DLP) {
      double e = S[N - 1], o = S[2 * N - 1];
#pragma unroll
      for (int k = N - 2; k >= 0; --k) e = fma(e, t, S[k]), o = fma(o, t, S[N + k]);
      a->sr = fma(w * z, e, a->sr);
      a->si = fma(w, o, a->si);
    }
    if constexpr (LAYER != BEM_SLP) {
      double e = S[3 * N - 1], o = S[4 * N - 1];
#pragma unroll
      for (int k = N - 2; k >= 0; --k) e = fma(e, t, S[2 * N + k]);
#pragma unroll
      for (int k = N - 2; k >= 1; --k) o = fma(o, t, S[3 * N + k]);
      const double ez = z3 * e;
      a->dr = fma(wd, ez, a->dr);
      a->di = fma(wd, o, a->di);
      if constexpr (MIRROR) a->mr = fma(wm, ez, a->mr), a->mi = fma(wm, o, a->mi);
    }
  } else {
    const double kr = kappa * r2 * z, wz = w * z, wd3 = wd * z3, wm3 = wm * z3;
    for (int k = 0; k < nr; ++k) {
      const double t = kr * R[k];
      double sn, cs;
      sincos_cw(t, &sn, &cs);
      if constexpr (LAYER != BEM_DLP) {
        const double c = wz * R[nr + k];
        a->sr = fma(c, cs, a->sr);
        a->si = fma(c, sn, a->si);
      }
      if constexpr (LAYER != BEM_SLP) {  // e^{i t} (1 - i t)
        const double v = R[2 * nr + k], fr = v * fma(t, sn, cs), fi = v * fma(-t, cs, sn);
        a->dr = fma(wd3, fr, a->dr);
        a->di = fma(wd3, fi, a->di);
        if constexpr (MIRROR) a->mr = fma(wm3, fr, a->mr), a->mi = fma(wm3, fi, a->mi);
      }
    }
  }
}

// Laplace: the radial moments; Helmholtz: the powers of kappa the series left.
template <int KERNEL, bool SER, class P>
__device__ __forceinline__ void ss_finish(const PairGeo &g, P S, double kappa, const SSSum &a,
                                          Acc<KERNEL> *vs, Acc<KERNEL> *vd, Acc<KERNEL> *vm) {
  if constexpr (KERNEL == BEM_LAPLACE) {
    vs->re = a.sr * S[0] * g.scale;
    vd->re = a.dr * S[2 * kSeries] * g.scale;
    vm->re = a.mr * S[2 * kSeries] * g.scale;
  } else {
    const double ks = SER ? kappa * g.scale : g.scale;
    const double kd = SER ? kappa * kappa * kappa * g.scale : g.scale;
    vs->re = a.sr * g.scale;
    vs->im = a.si * ks;
    vd->re = a.dr * g.scale;
    vd->im = a.di * kd;
    vm->re = a.mr * g.scale;
    vm->im = a.mi * kd;
  }
}

// One singular pair per lane over the directions [first, n) in steps of
// stride (P: a wave-uniform pointer when every lane takes all directions).
// U directions per step into U accumulators, written stage by stage so that
// the independent chains interleave; the sum order is fixed.
template <int KERNEL, int LAYER, bool MIRROR, bool VERTEX, bool SER, int U, class P>
__device__ __forceinline__ SSSum ss_sum(const PairGeo &g, P S, int n, int nr, double kappa,
                                        const double *m, int first, int stride) {
  const P T = S + 4 * kSeries, R = T + 5 * n;
  SSSum acc[U];
  int p = first;
  for (; p + (U - 1) * stride < n; p += U * stride) {
    double d[U][3], r2[U], h[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      ss_direction<VERTEX>(g, T, n, p + u * stride, d[u]);
      r2[u] = fma(d[u][0], d[u][0], fma(d[u][1], d[u][1], d[u][2] * d[u][2]));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) h[u] = __builtin_amdgcn_rsq(r2[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
      ss_add<KERNEL, LAYER, MIRROR, SER>(g, d[u], r2[u], h[u], T[4 * n + p + u * stride], S, R, nr,
                                         kappa, m, &acc[u]);
  }
  for (; p < n; p += stride) {
    double d[3];
    ss_direction<VERTEX>(g, T, n, p, d);
    const double r2 = fma(d[0], d[0], fma(d[1], d[1], d[2] * d[2]));
    ss_add<KERNEL, LAYER, MIRROR, SER>(g, d, r2, __builtin_amdgcn_rsq(r2), T[4 * n + p], S, R, nr,
                                       kappa, m, &acc[0]);
  }
#pragma unroll
  for (int u = 1; u < U; ++u) {
    acc[0].sr += acc[u].sr, acc[0].si += acc[u].si;
    acc[0].dr += acc[u].dr, acc[0].di += acc[u].di;
    acc[0].mr += acc[u].mr, acc[0].mi += acc[u].mi;
  }
  return acc[0];
}

// One singular pair per lane; all lanes of the wave share the class, so the
// tables are read with wave-uniform (scalar) loads.  LAYER = kSS: both layers
// (vs, vd), with MIRROR (vertex pairs) the double layer of (j, i) too (vm;
// ni: normal of tau_i).  Every sum takes the same operands in the same order
// whichever layers are asked for.  Bound by FP64 issue and, for the few pairs
// of a sub-tile, by the length of this one chain: about 30 (Laplace) to 70
// (Helmholtz, both layers) instructions per direction.  Against the sums over
// all q^3 eta points (q radial nodes each for Helmholtz, sine and cosine at
// each) the one-pass near field takes 0.79 -> 0.69 ms (8192 triangles,
// Laplace, q = 4) and 24.9 -> 22.3 ms (32768, Helmholtz, kappa = 4, q = 5).
template <int KERNEL, int LAYER, bool MIRROR = false>
__device__ __forceinline__ void ss_pair_lane(const PairGeo &g, const SSArgs &ss, int cls,
                                             double kappa, Acc<KERNEL> *vs, Acc<KERNEL> *vd,
                                             Acc<KERNEL> *vm = nullptr, const double *ni = nullptr) {
  constexpr int U = KERNEL == BEM_LAPLACE ? 4 : 2;
  const uniform_ptr S = (uniform_ptr)(pick4(ss.tab, cls));
  int n = pick4(ss.nd, cls);
  const int nr = pick4(ss.nr, cls);
  if (LAYER == BEM_DLP && cls == CLS_IDENTICAL) n = 0;  // <x - y, n> = 0 on one flat triangle
  Acc<KERNEL> none;
  const bool ser = KERNEL == BEM_LAPLACE || kappa * kappa * pair_extent2(g) <= 4.0;
  auto pass = [&](auto use_series) {
    constexpr bool SER = decltype(use_series)::value;
    SSSum a;
    if (cls == CLS_VERTEX) {
      a = ss_sum<KERNEL, LAYER, MIRROR, true, SER, U>(g, S, n, nr, kappa, ni, 0, 1);
    } else if (LAYER == kSS && cls == CLS_IDENTICAL) {
      a = ss_sum<KERNEL, BEM_SLP, false, false, SER, U>(g, S, n, nr, kappa, ni, 0, 1);
    } else {
      a = ss_sum<KERNEL, LAYER, false, false, SER, U>(g, S, n, nr, kappa, ni, 0, 1);
    }
    ss_finish<KERNEL, SER>(g, S, kappa, a, vs ? vs : &none, vd ? vd : &none, vm ? vm : &none);
  };
  if (ser) pass(std::true_type{});
  if constexpr (KERNEL == BEM_HELMHOLTZ) {
    if (!ser) pass(std::false_type{});
  }
}

// One singular pair per wave: lanes stride over the directions, then a
// butterfly sum.  Every lane returns the entry.
template <int KERNEL, int LAYER>
__device__ Acc<KERNEL> ss_pair_wave(const PairGeo &g, const SSArgs &ss, int cls, double kappa) {
  const int lane = threadIdx.x & (kWave - 1);
  const double *S = pick4(ss.tab, cls);
  int n = pick4(ss.nd, cls);
  const int nr = pick4(ss.nr, cls);
  if (LAYER == BEM_DLP && cls == CLS_IDENTICAL) n = 0;
  Acc<KERNEL> vs, vd, vm;
  auto pass = [&](auto use_series) {
    constexpr bool SER = decltype(use_series)::value;
    SSSum a = cls == CLS_VERTEX
                  ? ss_sum<KERNEL, LAYER, false, true, SER, 1>(g, S, n, nr, kappa, nullptr, lane, kWave)
                  : ss_sum<KERNEL, LAYER, false, false, SER, 1>(g, S, n, nr, kappa, nullptr, lane, kWave);
    if constexpr (LAYER == BEM_SLP) a.sr = wave_sum(a.sr);
    else a.dr = wave_sum(a.dr);
    if constexpr (KERNEL == BEM_HELMHOLTZ) {
      if constexpr (LAYER == BEM_SLP) a.si = wave_sum(a.si);
      else a.di = wave_sum(a.di);
    }
    ss_finish<KERNEL, SER>(g, S, kappa, a, &vs, &vd, &vm);
  };
  const bool ser = KERNEL == BEM_LAPLACE || kappa * kappa * pair_extent2(g) <= 4.0;  // uniform
  if (ser) pass(std::true_type{});
  if constexpr (KERNEL == BEM_HELMHOLTZ) {
    if (!ser) pass(std::false_type{});
  }
  return LAYER == BEM_SLP ? vs : vd;
}

}  // namespace dev
}  // namespace bem
