// Building blocks of the block assembly kernels (gfx950, wave64): LDS layout
// of a sub-tile and the sums of one regular entry, in FP64 and in FP32.
// Shared by the per-block, persistent and learned kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "bem_device.h"

namespace bem {
namespace blk {

using namespace dev;

constexpr uint16_t kNoPair = 0xffff; // empty slot of the sorted singular list
constexpr uint16_t kSwapped = 0x4000; // listed code: the mirror block's entry (j, i)
constexpr int kNearSingular = 0;     // list class of near-singular regular pairs (mixed)
constexpr int kSortPad = 512;        // room for the padding of up to 8 groups
constexpr int kBoth = 2;             // layer template value: single and double layer in one pass

// Row geometry in coordinates doubled and relative to the block's origin c,
// so that 1/r = h (3 - s h^2) with s = 4 r^2 and h ~ 1 / (2r).  A point of
// the triangle is x = V + (s/2) A + (e/2) B with s = xi, e = xi (eta - 1/2)
// in Duffy coordinates (xi, eta); with D = V - y
//   4 |x - y|^2 = |D|^2 + s <D, A> + e <D, B> + s^2 k0 + s e c1 + e^2 a22.
enum RowField {
  R_V,             // 2 (v0 - c)
  R_A = 3,         // 2 (2 e1 + e2)
  R_B = 6,         // 4 e2
  R_SG = 9,        // sqrt(g_i)
  R_C1, R_K0, R_A22,  // <A, B> / 2, |A|^2 / 4, |B|^2 / 4
  ROW_NF
};

// LDS layout of one sub-tile (up to TR rows x TC columns; triangle rule of nq
// points, room for nqp: rule_pad):
//   ys[nqp][TC]    column points (Y, w sqrt(g_j)): four doubles, Y = 2 (y - c);
//                  mixed: four floats, Y = 2 (y - v0_j) local to the triangle.
//                  Read as 16-byte words (broadcast in a wave).  The general sums
//                  and the learned form keep the column triangles instead,
//                  [kColumnFields][TC] doubles, the general sums then 4 |y_b -
//                  c_j|^2 of the points, [nq][TC] doubles (mixed: floats)
//   rg[ROW_NF][TR] row geometry
//   rule[3][nqp]   s, t, w of the triangle rule
//   cn[4][TC]      column normals n_j, <Y, n_j> (one value on the triangle's
//                  plane; mixed: unused)
//   cc[3][TC]      column centroids, doubled (Helmholtz phases)
//   both layers:   rn[3][TR] row normals
//   mixed only:    cg[3][TC] = 2 (v0_j - c); rb[6][TR], cb[6][TC] boxes
//   ints           rid[TR], rv[3][TR], cid[TC], cv[3][TC], count, bad, rcount, pad, per-group counts[16] and
//                  cursors[16] (classes at 0 .. 3, orders q at 8 + q)
//   list[slots]    uint16 codes (row | col << 6 | group << 12, kSwapped) of the pairs
//                  left to the FP64 pass (singular; near-singular if mixed),
//                  from the front; with per-entry orders, the regular pairs
//                  (group = order) from the back
//   sorted[slots + kSortPad]  codes grouped (by class or by order), each
//                  group padded to a multiple of 64 with kNoPair
struct Lds {
  double *ys, *rg, *rule, *cn, *cc, *rn, *cg, *rb, *cb;
  int *rid, *rv, *cid, *cv, *count, *bad, *rcount, *ccount, *cursor;
  uint16_t *list, *sorted;
};

__host__ __device__ __forceinline__ int ypoint_doubles(bool mixed) { return mixed ? 2 : 4; }

template <bool MIXED>
__device__ __forceinline__ Lds carve(double *base, const BlockArgs &a, bool both = false) {
  const int nqp = a.nq_pad, TR = a.tr, TC = a.tc;
  Lds l;
  l.ys = base;
  l.rg = l.ys + ypoint_doubles(MIXED) * nqp * TC;
  l.rule = l.rg + ROW_NF * TR;
  l.cn = l.rule + 3 * nqp;
  l.cc = l.cn + 4 * TC;
  l.rn = both ? l.cc + 3 * TC : nullptr;
  l.cg = l.cc + 3 * TC + (both ? 3 * TR : 0);
  l.rb = l.cg + (MIXED ? 3 * TC : 0);
  l.cb = l.rb + (MIXED ? 6 * TR : 0);
  int *ib = reinterpret_cast<int *>(l.cb + (MIXED ? 6 * TC : 0));
  l.rid = ib;
  l.rv = l.rid + TR;
  l.cid = l.rv + 3 * TR;
  l.cv = l.cid + TC;
  l.count = l.cv + 3 * TC;
  l.bad = l.count + 1;
  l.rcount = l.bad + 1;
  l.ccount = l.rcount + 2;
  l.cursor = l.ccount + 16;
  l.list = reinterpret_cast<uint16_t *>(l.cursor + 16);
  l.sorted = l.list + a.slots;
  return l;
}

// Whether triangle id may be in a block of short Helmholtz phases: kappa times
// the largest distance of a point from its centroid at most 3/4 (short_phase)
// and at least 1e-10 (coordinates are scaled by kappa then).
__device__ __forceinline__ bool is_brief(const BlockArgs &a, int id) {
  const double x = id >= 0 && id < a.nt ? a.kappa * a.kappa * a.geo[G_R2 * a.ldg + id] : 0.0;
  return x <= kShortPhase * kShortPhase && x >= 1e-20;
}

// ------------------------------------------------------------ regular sums
// Arithmetic of the two precisions.  FP64: 1/r from the hardware estimate and
// one Newton step, z = h u with u = 3 - s h^2.  FP32 (mixed form): the
// estimate h itself.  kInv: 1/r = kInv z for coordinates doubled (s = 4 r^2).
// Short phases take coordinates scaled by kappa kScale more, so that s u h
// (FP32: s h) is kappa r itself and 1/r = kappa kInvK z.
template <class T>
struct Arith;
template <>
struct Arith<double> {
  static constexpr double kInv = 1.0, kScale = 0.25, kInvK = 0.25;
  static __device__ __forceinline__ double mad(double a, double b, double c) { return __builtin_fma(a, b, c); }
  static __device__ __forceinline__ double rsq(double s) { return __builtin_amdgcn_rsq(s); }
  static __device__ __forceinline__ double newton(double s, double h) { return mad(-(s * h), h, 3.0); }
  static __device__ __forceinline__ double inv(double h, double u) { return h * u; }
  // h0 u0 + h1 u1
  static __device__ __forceinline__ double inv2(double h0, double u0, double h1, double u1) { return mad(h1, u1, h0 * u0); }
  static constexpr double kPhase = 0.25;  // kappa r = (kPhase kappa) s z, unscaled
  // factors of kappa r in scaled coordinates, and of a reference distance
  static __device__ __forceinline__ double phase(double t, double u) { return t * u; }
  static __device__ __forceinline__ double phase_from(double t, double u, double kr0) { return mad(t, u, -kr0); }
  static __device__ __forceinline__ double ref(double s) { return 2.0 * (s * rsq(s)); }
  static __device__ __forceinline__ void sincos(double x, double *s, double *c) { sincos_cw(x, s, c); }
  static __device__ __forceinline__ void sincos_short(double x, double *s, double *c) { short_phase(x, s, c); }
};
template <>
struct Arith<float> {
  static constexpr double kInv = 2.0, kScale = 0.5, kInvK = 1.0;
  static __device__ __forceinline__ float mad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
  static __device__ __forceinline__ float rsq(float s) { return __builtin_amdgcn_rsqf(s); }
  static __device__ __forceinline__ float newton(float, float) { return 1.0f; }
  static __device__ __forceinline__ float inv(float h, float) { return h; }
  static __device__ __forceinline__ float inv2(float h0, float, float h1, float) { return h0 + h1; }
  static constexpr double kPhase = 0.5;
  static __device__ __forceinline__ float phase(float s, float h) { return s * h; }
  static __device__ __forceinline__ float phase_from(float s, float h, float kr0) { return mad(s, h, -kr0); }
  static __device__ __forceinline__ float ref(float s) { return s * rsq(s); }
  static __device__ __forceinline__ void sincos(float x, float *s, float *c) { sincos_cw_f32(x, s, c); }
  static __device__ __forceinline__ void sincos_short(float x, float *s, float *c) { short_phase_f32(x, s, c); }
};

// One entry's operands: the row triangle (V relative to the column triangle's
// first vertex in the mixed form), the column's normal and centroid, the
// row's normal (both layers).
struct EntryGeo {
  double V[3], A[3], B[3], sg, c1, k0, a22;
  double n[3], yn;  // n_j, <Y, n_j>
  double m[3];      // n_i
  double cen[3];    // centroid of tau_j, doubled, in the coordinates of V
};

// Sums of an entry without the factor 1/(4 pi) (and 1/2 of the doubled normal
// distance): single layer, double layer, double layer of (j, i).
template <int KERNEL>
struct Sums {
  Acc<KERNEL> s, d, m;
};

// Column points from LDS (b-th point of the rule).
struct PointsLds64 {
  const double2 *p;
  int stride;
  struct P { double2 a, b; };
  __device__ __forceinline__ P get(int b) const { return {p[b * stride], p[b * stride + 1]}; }
  static __device__ __forceinline__ void unpack(const P &q, double *y, double *w) { y[0] = q.a.x, y[1] = q.a.y, y[2] = q.b.x, *w = q.b.y; }
};
struct PointsLds32 {
  const float4 *p;
  int stride;
  typedef float4 P;
  __device__ __forceinline__ P get(int b) const { return p[b * stride]; }
  static __device__ __forceinline__ void unpack(const P &q, float *y, float *w) { y[0] = q.x, y[1] = q.y, y[2] = q.z, *w = q.w; }
};

// Column points formed from the triangle in LDS (2 (v0 - origin), 2 e1, 2 e2,
// sqrt(g), a stride apart) and the rule r[3][n] read by scalar loads.
constexpr int kColumnFields = 10;
struct PointsOfRule {
  const double *c;
  int stride;
  uniform_ptr r;
  int n;
  struct P { double y[3], w; };
  __device__ __forceinline__ P get(int b) const {
    const double s = r[b], t = r[n + b];
    P p;
#pragma unroll
    for (int m = 0; m < 3; ++m)
      p.y[m] = fma(s, c[(3 + m) * stride], fma(t, c[(6 + m) * stride], c[m * stride]));
    p.w = r[2 * n + b] * c[9 * stride];
    return p;
  }
  static __device__ __forceinline__ void unpack(const P &q, double *y, double *w) { y[0] = q.y[0], y[1] = q.y[1], y[2] = q.y[2], *w = q.w; }
};

// The rule's constants in the precision of the sums, wave-uniform.
template <class T>
struct TablePtr {
  typedef const T __attribute__((address_space(4))) *type;
  static __device__ __forceinline__ type of(const double *t) { return (type)t; }
};

// Points of a column triangle for the general sums: the rule's coordinates
// from the centroid and weight (general_table, scalar loads) and 4 |y - c|^2
// from LDS.
template <class T>
struct PointsOfTriangle {
  const T *g;
  int stride;
  typename TablePtr<T>::type t;
  int n;
  struct P { T g, u, v, w; };
  __device__ __forceinline__ P get(int b) const { return {g[b * stride], t[4 * n + b], t[5 * n + b], t[2 * n + b]}; }
};

// Two points per step, the next one's LDS reads issued before the current
// one's arithmetic (no register copies between steps).
// ONE: one point per step with the copies (a third copy of a long body, for
// the last of an odd number of points, costs registers).
template <bool ONE, class PTS, class F>
__device__ __forceinline__ void for_points(const PTS &pts, int n, F &&point) {
  typename PTS::P a = pts.get(0);
  int k = 0;
  if constexpr (ONE) {
    for (; k < n; ++k) {
      const typename PTS::P b = pts.get(k + 1 < n ? k + 1 : n - 1);
      __builtin_amdgcn_sched_barrier(0);
      point(a);
      a = b;
    }
    return;
  }
  for (; k + 2 <= n; k += 2) {
    const typename PTS::P b = pts.get(k + 1);
    __builtin_amdgcn_sched_barrier(0);  // keep the reads ahead of the arithmetic
    point(a);
    a = pts.get(k + 2 < n ? k + 2 : n - 1);
    __builtin_amdgcn_sched_barrier(0);
    point(b);
  }
  if (k < n) point(a);
}

// Kernel values of one column point against x-points, summed with weights.
// Everything a point pair costs beyond its distance is here:
//   single layer  sum w k,   double layer  sum wn k3 (wn = w <X - Y, n_j>),
//   both layers   t1 = sum w k3, t2 = sum wn k3 and the single layer's sum,
// with k = 1/r, k3 = 1/r^3, times e^{i kappa r} resp. e^{i kappa r} (1 - i
// kappa r) for Helmholtz.  SHORT: phases relative to kr0 (kappa r - kr0 in
// [-3/4, 3/4]), the common factor e^{i kr0} left to the caller.
template <int KERNEL, int LAYER, class T>
struct PointSums {
  T sr = 0, si = 0, t1r = 0, t1i = 0, t2r = 0, t2i = 0;
};

// One x-point at squared distance s with estimate h: the single layer's value
// (kr_, ki_), the double layer's phase factor (fr, fi) and z^3 (Laplace: fr
// unused).
template <int KERNEL, int LAYER, bool SHORT, class T>
struct PairValue {
  typedef Arith<T> M;
  T kr_, ki_, fr, fi, z3, z, sn, cs;
  __device__ __forceinline__ void eval(T s, T h, T kq, T kr0) {
    if constexpr (KERNEL == BEM_LAPLACE) {
      z = M::inv(h, M::newton(s, h));
      kr_ = z;
      if constexpr (LAYER != BEM_SLP) z3 = z * z * z;
    } else {
      T kr = 0;
      if constexpr (SHORT) {
        T t, u;  // kappa r = t u
        if constexpr (std::is_same<T, double>::value) {
          t = s * h;
          u = M::mad(-t, h, (T)3);
          z = h * u;
        } else {
          t = s;
          u = z = h;
        }
        if constexpr (LAYER != BEM_SLP) {
          kr = M::phase(t, u);
          M::sincos_short(kr - kr0, &sn, &cs);
        } else {
          M::sincos_short(M::phase_from(t, u, kr0), &sn, &cs);
        }
      } else {
        z = M::inv(h, M::newton(s, h));
        kr = kq * s * z;
        M::sincos(kr, &sn, &cs);
      }
      if constexpr (LAYER != BEM_DLP) kr_ = z * cs, ki_ = z * sn;
      if constexpr (LAYER != BEM_SLP) {
        z3 = z * z * z;
        fr = M::mad(kr, sn, cs);
        fi = M::mad(-kr, cs, sn);
      }
    }
  }
  // the double layer's value, times z^3
  __device__ __forceinline__ T dr() const { return KERNEL == BEM_LAPLACE ? z3 : z3 * fr; }
  __device__ __forceinline__ T di() const { return z3 * fi; }
};

// Adds the value of one x-point at squared distance sq (estimate h of its
// reciprocal root) with weight w, w <X - Y, n_j> = wn.
template <int KERNEL, int LAYER, class T>
__device__ __forceinline__ void add_value(T sq, T h, T kq, T w, T wn, PointSums<KERNEL, LAYER, T> *ps) {
  typedef Arith<T> M;
  PairValue<KERNEL, LAYER, false, T> v;
  v.eval(sq, h, kq, (T)0);
  if constexpr (KERNEL == BEM_LAPLACE) {
    if constexpr (LAYER != BEM_DLP) ps->sr = M::mad(w, v.z, ps->sr);
    if constexpr (LAYER == kBoth) ps->t1r = M::mad(w, v.z3, ps->t1r);
    if constexpr (LAYER != BEM_SLP) ps->t2r = M::mad(wn, v.z3, ps->t2r);
  } else {
    // the weight goes to the factor that real and imaginary part share
    if constexpr (LAYER != BEM_DLP) {
      const T wz = w * v.z;
      ps->sr = M::mad(wz, v.cs, ps->sr), ps->si = M::mad(wz, v.sn, ps->si);
    }
    if constexpr (LAYER == BEM_DLP) {
      const T wz = wn * v.z3;
      ps->t2r = M::mad(wz, v.fr, ps->t2r), ps->t2i = M::mad(wz, v.fi, ps->t2i);
    } else if constexpr (LAYER == kBoth) {
      const T re = v.dr(), im = v.di();
      ps->t1r = M::mad(w, re, ps->t1r), ps->t1i = M::mad(w, im, ps->t1i);
      ps->t2r = M::mad(wn, re, ps->t2r), ps->t2i = M::mad(wn, im, ps->t2i);
    }
  }
}

// Adds one column point's sums, weighted: wy (entry), wm (transposed double
// layer), both rotated by e^{i kr0} = (cy, sy) when SHORT.
template <int KERNEL, int LAYER, bool SHORT, class T>
struct EntrySums {
  typedef Arith<T> M;
  T sr = 0, si = 0, dr = 0, di = 0, mr = 0, mi = 0;
  static __device__ __forceinline__ void rot(T w, T cy, T sy, T re, T im, T *ar, T *ai) {
    if constexpr (KERNEL == BEM_LAPLACE) {
      *ar = M::mad(w, re, *ar);
    } else if constexpr (!SHORT) {
      *ar = M::mad(w, re, *ar);
      *ai = M::mad(w, im, *ai);
    } else {
      const T cw = w * cy, sw = w * sy;
      *ar = M::mad(cw, re, M::mad(-sw, im, *ar));
      *ai = M::mad(cw, im, M::mad(sw, re, *ai));
    }
  }
  __device__ __forceinline__ void add(const PointSums<KERNEL, LAYER, T> &p, T wy, T wm, T cy, T sy) {
    if constexpr (LAYER != BEM_DLP) rot(wy, cy, sy, p.sr, p.si, &sr, &si);
    if constexpr (LAYER != BEM_SLP) rot(wy, cy, sy, p.t2r, p.t2i, &dr, &di);
    if constexpr (LAYER == kBoth) rot(wm, cy, sy, p.t1r, p.t1i, &mr, &mi);
  }
  // to FP64, times sqrt(g_i) and the powers of inv (1/r = inv z); SHORT:
  // rotated by e^{i kr00} = (c0, s0), conjugated for a negative kappa
  __device__ __forceinline__ void finish(double sg, double inv, double c0, double s0, bool neg,
                                         Sums<KERNEL> *o) const {
    auto put = [&](double f, T re, T im, Acc<KERNEL> *v) {
      const double r = f * (double)re;
      if constexpr (KERNEL == BEM_LAPLACE) {
        v->re = r;
      } else {
        const double i = f * (double)im;
        if constexpr (SHORT) {
          v->re = __builtin_fma(c0, r, -s0 * i);
          const double w = __builtin_fma(c0, i, s0 * r);
          v->im = neg ? -w : w;
        } else {
          v->re = r;
          v->im = i;
        }
      }
    };
    const double f1 = sg * inv, f3 = f1 * inv * inv;
    if constexpr (LAYER != BEM_DLP) put(f1, sr, si, &o->s);
    if constexpr (LAYER != BEM_SLP) put(f3, dr, di, &o->d);
    if constexpr (LAYER == kBoth) put(f3, mr, mi, &o->m);
  }
};

// Offsets in the table of a Duffy rule of order Q (duffy_table): per xi
// (xi, xi^2, w_xi xi, w_xi xi^2); the half-width nodes delta > 0 of eta =
// 1/2 +- delta, their squares, the eta weights w (pairs, then the centre of an
// odd order) and w delta of the pairs; for every (xi, pair) xi delta and
// (xi, eta) the full weight; and per xi c = xi - 2/3 and c^2.
template <int Q>
struct DuffyAt {
  static constexpr int H = Q / 2, HC = (Q + 1) / 2;
  static constexpr int J = 0, D = 4 * Q, D2 = D + H, W = D2 + H, WD = W + HC, XD = WD + H,
                       WF = XD + Q * H, CC = WF + Q * HC;
};

// Sums over the point pairs of one regular entry, Duffy rule of order Q on
// both triangles.  Bound by FP64 (FP32) issue, so the point pair is cut to
// what its own distance needs: on the row triangle the squared distance is a
// quadratic polynomial of the Duffy coordinates whose coefficients take 12
// operations per column point, then per xi two or three and per symmetric eta
// pair 1/2 +- delta three (2 to 2.4 per point pair, from 4 for coordinates of
// every x-point); equal weights of a pair are applied once, to its sum.  The
// rule's constants are wave-uniform (scalar registers).  FP32 takes the
// polynomial about the row's centroid, where its terms are a quarter as large
// (largest error of 64 x 64 sheets 0.03 triangle sizes apart, order 4: 1.4e-5 about
// the vertex, 1e-6 about the centroid, 5e-6 with plain coordinates).
// Every xi unrolled, products of constants and the double layer's point weights
// w <X - Y, n_j> (w (n0 + xi na +- xi delta nb)) kept: up to 72 of 229 registers
// for Laplace, no spills (a loop over xi instead, order 5 / 6: coupling of 6272
// triangles, double layer 3.36 / 6.76 -> 4.21 / 8.64 ms, single layer 1.41 / 3.13
// -> 1.62 / 3.23, one-pass near field 1.03 / 2.03 -> 1.17 / 2.18).  Helmholtz
// with the scheduling held to one xi (free, the chains of Q^2 sines and
// cosines spill); 4608 triangles, loop -> unrolled: coupling, double layer,
// order 3 / 4 / 5 / 6: 1.28 / 3.27 / 7.50 / 15.1 -> 1.16 / 3.06 / 7.09 / 14.4 ms,
// single layer 0.63 / 1.42 -> 0.57 / 1.39 and no gain from order 5 on (3.21,
// 6.64 -> 3.21, 6.67), one-pass near field, order 5: 2.44 -> 2.36.
// ROLL, the loop, where unrolling does not pay: Helmholtz single layer from
// order 5, and FP32 Helmholtz but for the double layer up to order 4 (single
// layer with general phases 2.19 -> 2.31 ms; one kernel for all layers, step of
// 3200 triangles with the double layer unrolled, order 5 / 6: 3.61 / 6.87 -> 3.73
// / 7.43).  There the double layer's weights are formed at every point pair
// (their terms summed separately: 4.20 -> 4.40 ms), or (both layers) their
// three terms are summed separately and combined per column point.
// Per point pair (FP64 instructions, v_rsq_f64 as four): Laplace single, double,
// both layers 12, 14, 16 -> 10.3, 12.8, 15.2; Helmholtz 46, 50, 55 -> 28, 34,
// 43 with short phases.  Vector units 95 % busy (18432 triangles, Helmholtz
// coupling): 38.6 -> 29.9 ms; Laplace coupling (8192, q = 4) 2.13 -> 1.82 ms,
// one-pass near field 0.69 -> 0.59 ms, Helmholtz (32768, q = 5) 22.3 -> 17.8 ms.
// FP64 and FP32 matrix instructions were no help: they do not overlap with the
// vector unit's (a 16 x 16 x 4 product takes the 64 cycles of its multiply-adds).
template <int KERNEL, int LAYER, int Q, bool SHORT, class T, class PTS>
__device__ __forceinline__ void duffy_sums(const EntryGeo &g, const double *table, double kappa,
                                           const PTS &pts, Sums<KERNEL> *out) {
  typedef Arith<T> M;
  typedef DuffyAt<Q> C;
  constexpr int H = C::H, HC = C::HC;
  constexpr bool ODD = Q & 1, HELM = KERNEL == BEM_HELMHOLTZ;
  constexpr bool FP64 = std::is_same<T, double>::value, CEN = !FP64;
  constexpr bool ROLL = HELM && (FP64 ? LAYER == BEM_SLP && Q >= 5 : LAYER != BEM_DLP || Q >= 5);
  constexpr bool LIN = ROLL && LAYER == kBoth;    // double-layer weights in three sums
  constexpr bool FLY = ROLL && LAYER == BEM_DLP;  // formed at every point pair
  const typename TablePtr<T>::type c = TablePtr<T>::of(table);
  // short phases: coordinates scaled by f so that kappa r needs no factor
  const double ka = fabs(kappa), f = HELM && SHORT ? ka * M::kScale : 1.0;
  // FP32: from the centroid V + A / 3 (xi = 2/3, eta = 1/2) instead of V
  const double third = CEN ? 1.0 / 3.0 : 0.0;
  const T V0 = (T)(f * fma(third, g.A[0], g.V[0])), V1 = (T)(f * fma(third, g.A[1], g.V[1])),
          V2 = (T)(f * fma(third, g.A[2], g.V[2]));
  const T A0 = (T)(f * g.A[0]), A1 = (T)(f * g.A[1]), A2 = (T)(f * g.A[2]);
  const T B0 = (T)(f * g.B[0]), B1 = (T)(f * g.B[1]), B2 = (T)(f * g.B[2]);
  const T c1 = (T)(f * f * g.c1), k0 = (T)(f * f * g.k0), a22 = (T)(f * f * g.a22), mf = (T)-f;
  // terms in xi alone: xi^2 K, from the centroid c^2 k0 + xi^2 K (unrolled: of
  // every point, kept)
  T K[HC], KC[CEN && !ROLL ? Q : 1][HC];
#pragma unroll
  for (int k = 0; k < HC; ++k) {
    const T base = CEN ? (T)0 : k0;
    K[k] = k < H ? M::mad(c[C::D2 + k], a22, base) : base;
  }
  if constexpr (CEN && !ROLL) {
#pragma unroll
    for (int j = 0; j < Q; ++j)
#pragma unroll
      for (int k = 0; k < HC; ++k) KC[j][k] = M::mad(c[4 * j + 1], K[k], c[C::CC + 2 * j + 1] * k0);
  }
  T WN[ROLL ? 1 : Q][Q], n0 = 0, na = 0, nb = 0;
  if constexpr (LAYER != BEM_SLP) {
    n0 = (T)(fma(g.V[0], g.n[0], fma(g.V[1], g.n[1], g.V[2] * g.n[2])) - g.yn);
    na = (T)(0.5 * fma(g.A[0], g.n[0], fma(g.A[1], g.n[1], g.A[2] * g.n[2])));
    nb = (T)(0.5 * fma(g.B[0], g.n[0], fma(g.B[1], g.n[1], g.B[2] * g.n[2])));
  }
  if constexpr (LAYER != BEM_SLP && !ROLL) {
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const T base = M::mad(c[4 * j], na, n0);
#pragma unroll
      for (int k = 0; k < H; ++k) {
        const T e = c[C::XD + j * H + k] * nb;
        WN[j][2 * k] = c[C::WF + j * HC + k] * (base + e);
        WN[j][2 * k + 1] = c[C::WF + j * HC + k] * (base - e);
      }
      if (ODD) WN[j][Q - 1] = c[C::WF + j * HC + H] * base;
    }
  }
  T NB[H];
  if constexpr (FLY) {
#pragma unroll
    for (int k = 0; k < H; ++k) NB[k] = c[C::D + k] * nb;
  }
  T m0 = 0, m1 = 0, m2 = 0;
  if constexpr (LAYER == kBoth) {
    const double r = HELM && SHORT ? 1.0 / f : 1.0;
    m0 = (T)(r * g.m[0]), m1 = (T)(r * g.m[1]), m2 = (T)(r * g.m[2]);
  }
  const T kq = (T)(M::kPhase * kappa);
  T kr00 = 0;
  double c0 = 1.0, s0 = 0.0;
  if constexpr (HELM && SHORT) {
    // kappa times the distance of the centroids
    double r2 = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double d = fma(1.0 / 3.0, g.A[k], g.V[k]) - g.cen[k];
      r2 = fma(d, d, r2);
    }
    kr00 = (T)(0.5 * ka * (r2 * rsqrt_newton(r2)));
    sincos_cw((double)kr00, &s0, &c0);
  }
  EntrySums<KERNEL, LAYER, SHORT, T> sum;
  for_points<HELM>(pts, Q * Q, [&](const typename PTS::P &pt) {
    T y[3], wy;
    PTS::unpack(pt, y, &wy);
    const T D0 = M::mad(mf, y[0], V0), D1 = M::mad(mf, y[1], V1), D2 = M::mad(mf, y[2], V2);
    const T U = M::mad(D0, D0, M::mad(D1, D1, D2 * D2));
    const T R = M::mad(D0, A0, M::mad(D1, A1, D2 * A2));
    const T S = M::mad(D0, B0, M::mad(D1, B1, D2 * B2));
    T kr0 = 0, cy = 1, sy = 0;
    if constexpr (HELM && SHORT) {
      // the row centroid (xi = 2/3, eta = 1/2); only the reference of the
      // phases, so the hardware estimate serves
      const T q0 = CEN ? U : M::mad((T)(4.0 / 9.0), k0, M::mad((T)(2.0 / 3.0), R, U));
      kr0 = M::ref(q0);
      M::sincos_short(kr0 - kr00, &sy, &cy);
    }
    PointSums<KERNEL, LAYER, T> ps;
    T txr = 0, txi = 0, tbr = 0, tbi = 0;  // LIN: xi and xi delta moments
    // the q points of one xi (x, from the centroid xc), weight wx; j: its index
    // if unrolled
    auto row = [&](int j, T x, T x2, T wx, T wxx, T xc, T xc2) {
      T E = M::mad(xc, R, U);
      if (CEN && ROLL) E = M::mad(xc2, k0, E);
      T O = M::mad(xc, c1, S);
      if (ROLL) O *= x;
      auto middle = [&](int k) -> T {
        if constexpr (CEN && !ROLL) return E + KC[j][k];
        else return CEN && k >= H ? E : M::mad(x2, K[k], E);
      };
      T s[Q], h[Q];
#pragma unroll
      for (int k = 0; k < H; ++k) {
        const T mid = middle(k);
        const T dl = ROLL ? c[C::D + k] : c[C::XD + j * H + k];
        s[2 * k] = M::mad(dl, O, mid);
        s[2 * k + 1] = M::mad(-dl, O, mid);
      }
      if (ODD) s[Q - 1] = middle(HC - 1);
#pragma unroll
      for (int k = 0; k < Q; ++k) h[k] = M::rsq(s[k]);
      // weighted sums over eta: into the point's sums (full weights) or first
      // into this xi's
      PointSums<KERNEL, LAYER, T> in;
      T ibr = 0, ibi = 0;
      const T base = FLY ? M::mad(x, na, n0) : (T)0;
      PointSums<KERNEL, LAYER, T> &w = ROLL ? in : ps;
      auto wt = [&](int k) { return ROLL ? c[C::W + k] : c[C::WF + j * HC + k]; };
      if constexpr (KERNEL == BEM_LAPLACE && LAYER == BEM_SLP) {
#pragma unroll
        for (int k = 0; k < H; ++k)
          w.sr = M::mad(wt(k), M::inv2(h[2 * k], M::newton(s[2 * k], h[2 * k]), h[2 * k + 1],
                                       M::newton(s[2 * k + 1], h[2 * k + 1])), w.sr);
        if (ODD) w.sr = M::mad(wt(H), M::inv(h[Q - 1], M::newton(s[Q - 1], h[Q - 1])), w.sr);
      } else {
#pragma unroll
        for (int k = 0; k < HC; ++k) {
          const bool two = k < H;
          const int a = two ? 2 * k : Q - 1;
          PairValue<KERNEL, LAYER, SHORT, T> v, u;
          v.eval(s[a], h[a], kq, kr0);
          if (two) u.eval(s[a + 1], h[a + 1], kq, kr0);
          if constexpr (LAYER != BEM_DLP) {
            w.sr = M::mad(wt(k), two ? v.kr_ + u.kr_ : v.kr_, w.sr);
            if constexpr (HELM) w.si = M::mad(wt(k), two ? v.ki_ + u.ki_ : v.ki_, w.si);
          }
          if constexpr (FLY) {
            const T wa = two ? M::mad(x, NB[k], base) * v.z3 : base * v.z3;
            const T wb = two ? M::mad(-x, NB[k], base) * u.z3 : (T)0;
            if constexpr (HELM) {
              const T pr = wa * v.fr, pi = wa * v.fi;
              w.t2r = M::mad(wt(k), two ? M::mad(wb, u.fr, pr) : pr, w.t2r);
              w.t2i = M::mad(wt(k), two ? M::mad(wb, u.fi, pi) : pi, w.t2i);
            } else {
              w.t2r = M::mad(wt(k), two ? wa + wb : wa, w.t2r);
            }
          } else if constexpr (LAYER != BEM_SLP) {
            const T ar = v.dr(), br = two ? u.dr() : (T)0;
            T ai = 0, bi = 0;
            if constexpr (HELM) ai = v.di(), bi = two ? u.di() : (T)0;
            if constexpr (LAYER == kBoth) {
              w.t1r = M::mad(wt(k), two ? ar + br : ar, w.t1r);
              if constexpr (HELM) w.t1i = M::mad(wt(k), two ? ai + bi : ai, w.t1i);
            }
            if constexpr (LIN) {
              if (two) {
                ibr = M::mad(c[C::WD + k], ar - br, ibr);
                if constexpr (HELM) ibi = M::mad(c[C::WD + k], ai - bi, ibi);
              }
            } else {
              ps.t2r = M::mad(WN[ROLL ? 0 : j][a], ar, ps.t2r);
              if (two) ps.t2r = M::mad(WN[ROLL ? 0 : j][a + 1], br, ps.t2r);
              if constexpr (HELM) {
                ps.t2i = M::mad(WN[ROLL ? 0 : j][a], ai, ps.t2i);
                if (two) ps.t2i = M::mad(WN[ROLL ? 0 : j][a + 1], bi, ps.t2i);
              }
            }
          }
        }
      }
      if constexpr (ROLL) {
        if constexpr (LAYER != BEM_DLP) {
          ps.sr = M::mad(wx, in.sr, ps.sr);
          if constexpr (HELM) ps.si = M::mad(wx, in.si, ps.si);
        }
        if constexpr (FLY) {
          ps.t2r = M::mad(wx, in.t2r, ps.t2r);
          if constexpr (HELM) ps.t2i = M::mad(wx, in.t2i, ps.t2i);
        }
        if constexpr (LIN) {
          ps.t1r = M::mad(wx, in.t1r, ps.t1r);
          if constexpr (HELM) ps.t1i = M::mad(wx, in.t1i, ps.t1i);
          txr = M::mad(wxx, in.t1r, txr);
          tbr = M::mad(wxx, ibr, tbr);
          if constexpr (HELM) {
            txi = M::mad(wxx, in.t1i, txi);
            tbi = M::mad(wxx, ibi, tbi);
          }
        }
      }
    };
    if constexpr (ROLL) {
      // the next xi's constants are read before this one's arithmetic
      T x = c[0], x2 = c[1], wx = c[2], wxx = c[3], xc = x, xc2 = x2;
      if (CEN) xc = c[C::CC], xc2 = c[C::CC + 1];
#pragma unroll 1
      for (int j = 0; j < Q; ++j) {
        const int n = j + 1 < Q ? j + 1 : j, p = 4 * n;
        const T nx = c[p], nx2 = c[p + 1], nwx = c[p + 2], nwxx = c[p + 3];
        const T nc = CEN ? c[C::CC + 2 * n] : nx, nc2 = CEN ? c[C::CC + 2 * n + 1] : nx2;
        row(0, x, x2, wx, wxx, xc, xc2);
        x = nx, x2 = nx2, wx = nwx, wxx = nwxx, xc = nc, xc2 = nc2;
      }
    } else {
#pragma unroll
      for (int j = 0; j < Q; ++j) {
        row(j, c[4 * j], c[4 * j + 1], (T)0, (T)0, c[CEN ? C::CC + 2 * j : 4 * j], (T)0);
        // one xi's chains at a time: scheduled across, they spill
        if constexpr (HELM) __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (LIN) {
      ps.t2r = M::mad(n0, ps.t1r, M::mad(na, txr, nb * tbr));
      if constexpr (HELM) ps.t2i = M::mad(n0, ps.t1i, M::mad(na, txi, nb * tbi));
    }
    T wm = 0;
    // wy 2 <y - x, n_i>: <X, n_i> is one value on the row triangle's plane
    if constexpr (LAYER == kBoth) wm = -wy * M::mad(D0, m0, M::mad(D1, m1, D2 * m2));
    sum.add(ps, wy, wm, cy, sy);
  });
  sum.finish(g.sg, HELM && SHORT ? ka * M::kInvK : M::kInv, c0, s0, kappa < 0.0, out);
}

// The same for any triangle rule (general_table, in T and in FP64), x-points in register chunks
// of XC (zero weights and the last point repeated past the end).  With X0 twice
// the difference of the centroids, x = c_i + (s/2) A + (e/2) B, E = 2 e_j and s, u,
// v counted from the centroids the squared distance is a polynomial of the rule
// coordinates of both triangles,
//   4 |x - y|^2 = |X0|^2 + s <X0, A> + e <X0, B> + s^2 k0 + s e c1 + e^2 a22
//     - u <2 X0 + s A + e B, E1> - v <2 X0 + s A + e B, E2> + |u E1 + v E2|^2:
// nine coefficients of the pair, nine operations per x-point for its three
// in (1, u, v), one number per column point from LDS, three operations per point
// pair.  (Quadratic in the row's coordinates alone, each column point took twelve
// per chunk.)
// The chunks' sums are added in FP64: in the mixed form the FP32 sums are no
// longer than the rule, whatever the chunk.
// Against four operations per pair on coordinates of every x-point in chunks of
// 8, 9, 7, 5 or 4 (Laplace, double layer, coupling; 3200 triangles orders 7 and 8,
// 2048 above): 5.77 -> 5.53 ms, 9.61 -> 9.12, order 9 10.0 -> 7.5, order 12 33.6 ->
// 23.3; the matrix step of 1152 triangles, order 8 / 9 / 12: 6.3 / 9.7 / 31.1 ->
// 6.0 / 9.3 / 30.2.
template <int KERNEL, int LAYER, int XC, class T>
__device__ __forceinline__ void general_sums(const EntryGeo &g, const double *col, const T *gb, int TC,
                                             const double *table, const double *table64, int nq,
                                             double kappa, Sums<KERNEL> *out) {
  typedef Arith<T> M;
  const typename TablePtr<T>::type c = TablePtr<T>::of(table);
  const uniform_ptr d = (uniform_ptr)table64;
  auto dot = [](const T *a, const T *b) { return M::mad(a[0], b[0], M::mad(a[1], b[1], a[2] * b[2])); };
  T X[3], A[3], B[3], E1[3], E2[3];
  double c0 = 0, n0 = 0, ns = 0, nt = 0, m0 = 0, m1 = 0, m2 = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double x = fma(1.0 / 3.0, g.A[k], g.V[k]) - g.cen[k];
    const double f1 = col[(3 + k) * TC], f2 = col[(6 + k) * TC];
    X[k] = (T)x, A[k] = (T)g.A[k], B[k] = (T)g.B[k], E1[k] = (T)f1, E2[k] = (T)f2;
    c0 = fma(x, x, c0);  // its rounding is in every point pair: in FP64
    if constexpr (LAYER != BEM_SLP)
      n0 = fma(g.V[k], g.n[k], n0), ns = fma(fma(-0.25, g.B[k], 0.5 * g.A[k]), g.n[k], ns), nt = fma(0.5 * g.B[k], g.n[k], nt);
    if constexpr (LAYER == kBoth) m0 = fma(-x, g.m[k], m0), m1 = fma(f1, g.m[k], m1), m2 = fma(f2, g.m[k], m2);
  }
  n0 -= g.yn;
  const T C0 = (T)c0, K0 = (T)g.k0, C1 = (T)g.c1, A22 = (T)g.a22;
  const T ra = dot(X, A), rb = dot(X, B);
  const T p0 = (T)-2 * dot(X, E1), pa = -dot(A, E1), pb = -dot(B, E1);
  const T q0 = (T)-2 * dot(X, E2), qa = -dot(A, E2), qb = -dot(B, E2);
  const T M0 = (T)m0, M1 = (T)m1, M2 = (T)m2;  // 2 <y - x, n_i> = m0 + u m1 + v m2
  const T kq = (T)(M::kPhase * kappa);
  const PointsOfTriangle<T> pts{gb, TC, c, nq};
  EntrySums<KERNEL, LAYER, false, double> total;
  for (int ch = 0; ch < nq; ch += XC) {
    EntrySums<KERNEL, LAYER, false, T> sum;
    T r[XC], p[XC], q[XC], W[XC], WN[XC];
#pragma unroll
    for (int a = 0; a < XC; ++a) {
      const int k = min(ch + a, nq - 1);
      const T s = c[4 * nq + k], e = c[3 * nq + k];
      r[a] = M::mad(c[6 * nq + k], K0, M::mad(c[7 * nq + k], C1, M::mad(c[8 * nq + k], A22, M::mad(s, ra, M::mad(e, rb, C0)))));
      p[a] = M::mad(s, pa, M::mad(e, pb, p0));
      q[a] = M::mad(s, qa, M::mad(e, qb, q0));
      W[a] = ch + a < nq ? c[2 * nq + k] : (T)0;
      if constexpr (LAYER != BEM_SLP)
        WN[a] = ch + a < nq ? (T)(d[2 * nq + k] * fma(d[k], ns, fma(d[nq + k], nt, n0))) : (T)0;
    }
    for_points<KERNEL == BEM_HELMHOLTZ>(pts, nq, [&](const typename PointsOfTriangle<T>::P &y) {
      T sq[XC], h[XC];
#pragma unroll
      for (int a = 0; a < XC; ++a) sq[a] = M::mad(y.v, q[a], M::mad(y.u, p[a], r[a] + y.g));
#pragma unroll
      for (int a = 0; a < XC; ++a) h[a] = M::rsq(sq[a]);
      PointSums<KERNEL, LAYER, T> ps;
#pragma unroll
      for (int a = 0; a < XC; ++a) add_value(sq[a], h[a], kq, W[a], WN[a], &ps);
      T wm = 0;
      if constexpr (LAYER == kBoth) wm = y.w * M::mad(y.v, M2, M::mad(y.u, M1, M0));
      sum.add(ps, y.w, wm, (T)1, (T)0);
    });
    total.sr += sum.sr, total.si += sum.si;
    total.dr += sum.dr, total.di += sum.di;
    total.mr += sum.mr, total.mi += sum.mi;
  }
  total.finish(g.sg * col[9 * TC], M::kInv, 1.0, 0.0, false, out);
}

// The same for the seven-point rule, whose pairs are too few for the general
// sums' coefficients (coupling of 10368 triangles, Laplace single / double layer:
// 888 / 1135 us with them, 737 / 870 so, 837 / 953 with three differences per
// point pair): all x-points in registers, the distance a polynomial of the row's
// rule coordinates alone.  Helmholtz is bound by its sines and cosines: 1946 /
// 2140 us, 1945 / 2132.
template <int KERNEL, int LAYER, class T, class PTS>
__device__ __forceinline__ void seven_sums(const EntryGeo &g, const double *table, const double *table64,
                                           double kappa, const PTS &pts, Sums<KERNEL> *out) {
  typedef Arith<T> M;
  constexpr int XC = 7;
  const typename TablePtr<T>::type c = TablePtr<T>::of(table);
  const uniform_ptr d = (uniform_ptr)table64;
  // from the row's centroid
  const T V0 = (T)fma(1.0 / 3.0, g.A[0], g.V[0]), V1 = (T)fma(1.0 / 3.0, g.A[1], g.V[1]),
          V2 = (T)fma(1.0 / 3.0, g.A[2], g.V[2]);
  const T A0 = (T)g.A[0], A1 = (T)g.A[1], A2 = (T)g.A[2];
  const T B0 = (T)g.B[0], B1 = (T)g.B[1], B2 = (T)g.B[2];
  T m0 = 0, m1 = 0, m2 = 0;
  if constexpr (LAYER == kBoth) m0 = (T)g.m[0], m1 = (T)g.m[1], m2 = (T)g.m[2];
  // 2 <x - y, n_j> = n0 + s ns + t nt: often far below 2 |x - y|, in FP64
  double n0 = 0, ns = 0, nt = 0;
  if constexpr (LAYER != BEM_SLP) {
    n0 = fma(g.V[0], g.n[0], fma(g.V[1], g.n[1], g.V[2] * g.n[2])) - g.yn;
    nt = 0.5 * fma(g.B[0], g.n[0], fma(g.B[1], g.n[1], g.B[2] * g.n[2]));
    ns = fma(-0.5, nt, 0.5 * fma(g.A[0], g.n[0], fma(g.A[1], g.n[1], g.A[2] * g.n[2])));
  }
  const T kq = (T)(M::kPhase * kappa);
  T q[XC], WN[XC];
#pragma unroll
  for (int a = 0; a < XC; ++a) {
    q[a] = (T)fma(d[6 * XC + a], g.k0, fma(d[7 * XC + a], g.c1, d[8 * XC + a] * g.a22));
    if constexpr (LAYER != BEM_SLP) WN[a] = (T)(d[2 * XC + a] * fma(d[a], ns, fma(d[XC + a], nt, n0)));
  }
  EntrySums<KERNEL, LAYER, false, T> sum;
  for_points<false>(pts, XC, [&](const typename PTS::P &pt) {
    T y[3], wy;
    PTS::unpack(pt, y, &wy);
    const T D0 = V0 - y[0], D1 = V1 - y[1], D2 = V2 - y[2];
    const T U = M::mad(D0, D0, M::mad(D1, D1, D2 * D2));
    const T R = M::mad(D0, A0, M::mad(D1, A1, D2 * A2));
    const T S = M::mad(D0, B0, M::mad(D1, B1, D2 * B2));
    T sq[XC], h[XC];
#pragma unroll
    for (int a = 0; a < XC; ++a) sq[a] = M::mad(c[3 * XC + a], S, M::mad(c[4 * XC + a], R, U + q[a]));
#pragma unroll
    for (int a = 0; a < XC; ++a) h[a] = M::rsq(sq[a]);
    PointSums<KERNEL, LAYER, T> ps;
#pragma unroll
    for (int a = 0; a < XC; ++a)
      add_value(sq[a], h[a], kq, c[2 * XC + a], LAYER != BEM_SLP ? WN[a] : (T)0, &ps);
    T wm = 0;
    if constexpr (LAYER == kBoth) wm = -wy * M::mad(D0, m0, M::mad(D1, m1, D2 * m2));
    sum.add(ps, wy, wm, (T)1, (T)0);
  });
  sum.finish(g.sg, M::kInv, 1.0, 0.0, false, out);
}

// Rule variants of the kernels: the Duffy orders 2 .. 6, seven points, else the
// general sums in chunks of 4, 7, 8 or 9 x-points (rule_variant).
constexpr int kSeven = 13, kRule4 = 14, kRule7 = 17, kRule8 = 18, kRule9 = 19;

// Operands of entry (rl, cl) of the staged sub-tile.
template <int LAYER, bool MIXED>
__device__ __forceinline__ EntryGeo entry_geo(const Lds &l, int TR, int TC, int rl, int cl) {
  EntryGeo g;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    g.V[c] = l.rg[(R_V + c) * TR + rl];
    if (MIXED) g.V[c] -= l.cg[c * TC + cl];  // relative to the column triangle's first vertex
    g.A[c] = l.rg[(R_A + c) * TR + rl];
    g.B[c] = l.rg[(R_B + c) * TR + rl];
    g.n[c] = LAYER == BEM_SLP ? 0.0 : l.cn[c * TC + cl];
    g.m[c] = LAYER == kBoth ? l.rn[c * TR + rl] : 0.0;
    g.cen[c] = l.cc[c * TC + cl];
    if (MIXED) g.cen[c] -= l.cg[c * TC + cl];
  }
  g.yn = LAYER == BEM_SLP || MIXED ? 0.0 : l.cn[3 * TC + cl];
  g.sg = l.rg[R_SG * TR + rl];
  g.c1 = l.rg[R_C1 * TR + rl];
  g.k0 = l.rg[R_K0 * TR + rl];
  g.a22 = l.rg[R_A22 * TR + rl];
  return g;
}

// All sums of regular entry (rl, cl), FP64 or (mixed) FP32.  brief: Helmholtz
// with short phases, uniform in the workgroup (block_is_brief).
template <int KERNEL, int LAYER, int RULE, bool MIXED>
__device__ __forceinline__ void regular_sums(const Lds &l, int TR, int TC, int nq, int rl, int cl,
                                             const double *table, const double *table64, double kappa, bool brief, Sums<KERNEL> *o) {
  const EntryGeo g = entry_geo<LAYER, MIXED>(l, TR, TC, rl, cl);
  typedef typename std::conditional<MIXED, float, double>::type T;
  if constexpr (RULE >= kRule4) {
    const T *gb = reinterpret_cast<const T *>(l.ys + kColumnFields * TC);
    general_sums<KERNEL, LAYER, RULE - 10, T>(g, l.ys + cl, gb + cl, TC, table, table64, nq, kappa, o);
  } else {
    typename std::conditional<MIXED, PointsLds32, PointsLds64>::type pts;
    if constexpr (MIXED) {
      pts.p = reinterpret_cast<const float4 *>(l.ys) + cl;
      pts.stride = TC;
    } else {
      pts.p = reinterpret_cast<const double2 *>(l.ys) + 2 * cl;
      pts.stride = 2 * TC;
    }
    if constexpr (RULE == kSeven) seven_sums<KERNEL, LAYER, T>(g, table, table64, kappa, pts, o);
    else if (KERNEL == BEM_HELMHOLTZ && brief) duffy_sums<KERNEL, LAYER, RULE, true, T>(g, table, kappa, pts, o);
    else duffy_sums<KERNEL, LAYER, RULE, false, T>(g, table, kappa, pts, o);
  }
}

}  // namespace blk
}  // namespace bem
