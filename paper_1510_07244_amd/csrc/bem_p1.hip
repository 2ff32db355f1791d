// Piecewise-linear (P1) bases (Sec. 2.2, eq. reference_integral: the
// transformed basis functions are low-order polynomials).  For a pair of
// triangles the 3 x 3 local matrix
//     L_ab = int_{tau_i} int_{tau_j} lambda_a(x) k(x, y) mu_b(y) dy dx
// (lambda_a, mu_b the nodal functions of the triangles' vertices in mesh
// order) comes from the same rules as the piecewise-constant entries: on
// the reference triangle of Phi(s, t) = v0 + s e1 + t e2 the barycentric
// coordinates are (1 - s, s - t, t), so every rule point adds its weighted
// kernel value times the nine products of shape-function values.  The
// Galerkin matrix of the vertices is then the sum of the local matrices over
// the triangles around each vertex pair (k_p1_gather, a fixed-order gather
// in place of a scatter-add, so results are reproducible bit for bit).
#include <hip/hip_runtime.h>

#include "bem_device.h"

namespace bem {
namespace {

using namespace dev;

// Nine sums in the pair's own vertex order (relabelled for singular pairs)
// and where each of its rows / columns goes in mesh order.
template <int KERNEL>
struct Acc9 {
  double re[9], im[9];
  int pr[3], pc[3];
};

// kernel value k(x, y) for d = x - y (r = |d|), n the normal of tau_j;
// Helmholtz as (re, im)
template <int KERNEL, int LAYER>
__device__ __forceinline__ void kernel_value(double dx, double dy, double dz, const double *n,
                                             double kappa, double *kre, double *kim) {
  const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
  const double iz = rsqrt_newton(r2);
  double base = iz;
  if constexpr (LAYER == BEM_DLP) base = fma(dx, n[0], fma(dy, n[1], dz * n[2])) * iz * iz * iz;
  if constexpr (KERNEL == BEM_LAPLACE) {
    *kre = base;
    *kim = 0.0;
  } else {
    const double kr = kappa * r2 * iz;
    double sn, cs;
    sincos_cw(kr, &sn, &cs);
    if constexpr (LAYER == BEM_SLP) {
      *kre = base * cs;
      *kim = base * sn;
    } else {  // e^{ikr} (1 - i kr)
      *kre = base * fma(kr, sn, cs);
      *kim = base * fma(-kr, cs, sn);
    }
  }
}

// Regular pair by the triangle rule of each triangle: for every x-point of
// this lane (sub of G) the sums over the column points times 1, u and v give
// those of the three column shape functions, then the row point's three.
template <int KERNEL, int LAYER, int XC>
__device__ void p1_regular(const P1Args &a, int i, int j, int sub, int G, Acc9<KERNEL> *L) {
  for (int e = 0; e < 9; ++e) L->re[e] = L->im[e] = 0.0;
  for (int k = 0; k < 3; ++k) L->pr[k] = L->pc[k] = k;
  const int nq = a.nq;
  regular_rows<KERNEL, LAYER, false, true, XC>(a.geo, a.ldg, a.rule, nq, a.kappa, i, j, sub, G,
                                               [&](int p, double w, const RowSum &r) {
    const double *re = LAYER == BEM_SLP ? r.sr : r.dr, *im = LAYER == BEM_SLP ? r.si : r.di;
    const double s = a.rule[p], t = a.rule[nq + p];
    const double la[3] = {w * (1.0 - s), w * (s - t), w * t};
    const double br[3] = {re[0] - re[1], re[1] - re[2], re[2]};
    const double bi[3] = {im[0] - im[1], im[1] - im[2], im[2]};
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        L->re[3 * k + b] = fma(la[k], br[b], L->re[3 * k + b]);
        if constexpr (KERNEL == BEM_HELMHOLTZ) L->im[3 * k + b] = fma(la[k], bi[b], L->im[3 * k + b]);
      }
  });
  const double *g = a.geo;
  const double sc = g[G_SG * a.ldg + i] * g[G_SG * a.ldg + j] * kInv4Pi;
  for (int e = 0; e < 9; ++e) L->re[e] *= sc, L->im[e] *= sc;
}

// Singular pair by the Sauter-Schwab rule of its class (one wave per pair,
// lanes over the eta points; every xi node of the rule per eta point).
// After relabelling both maps start at a common vertex, so x - y = xi d(eta)
// with d = g1 E1_i + g2 E2_i - g3 E1_j - g4 E2_j; the shape functions are
// those of the relabelled vertices, summed into the mesh-order slots.
template <int KERNEL, int LAYER>
__device__ void p1_singular(const P1Args &a, int i, int j, int cls, Acc9<KERNEL> *L) {
  const int lane = threadIdx.x & (kWave - 1);
  for (int e = 0; e < 9; ++e) L->re[e] = L->im[e] = 0.0;
  const int *ti = a.tri + 3 * (int64_t)i, *tj = a.tri + 3 * (int64_t)j;
  int li[3], lj[3];
  relabel(ti[0], ti[1], ti[2], tj[0], tj[1], tj[2], cls, li, lj);
  for (int k = 0; k < 3; ++k) {  // mesh-order slot of relabelled vertex k
    L->pr[k] = ti[0] == li[k] ? 0 : (ti[1] == li[k] ? 1 : 2);
    L->pc[k] = tj[0] == lj[k] ? 0 : (tj[1] == lj[k] ? 1 : 2);
  }
  PairGeo pg;
  if (!pair_geometry(a.v, a.tri, a.nv, a.geo, a.ldg, i, j, cls, a.flags, &pg)) return;
  if (!(LAYER == BEM_DLP && cls == CLS_IDENTICAL)) {  // else <x - y, n> = 0: all zero
    const double *T = pick4(a.ss.eta, cls);  // full tables (the identical one too)
    const int np = pick4(a.ss.np, cls), q = a.ss.q;
    const double *X = a.ss.xi;  // [xi | w xi^2 | w xi | ...]
    for (int p = lane; p < np; p += kWave) {
      const double g1 = T[p], g2 = T[np + p], g3 = T[2 * np + p], g4 = T[3 * np + p];
      const double wt = T[4 * np + p];
      double d[3];
#pragma unroll
      for (int c = 0; c < 3; ++c)
        d[c] = fma(g1, pg.E1i[c], fma(g2, pg.E2i[c], fma(-g3, pg.E1j[c], -g4 * pg.E2j[c])));
      for (int k = 0; k < q; ++k) {
        const double xi = X[k];
        const double w = wt * xi * X[q + k];  // eta weight x w_a xi_a^3
        double kre, kim;
        kernel_value<KERNEL, LAYER>(xi * d[0], xi * d[1], xi * d[2], pg.n, a.kappa, &kre, &kim);
        const double lx[3] = {1.0 - xi * g1, xi * (g1 - g2), xi * g2};
        const double ly[3] = {1.0 - xi * g3, xi * (g3 - g4), xi * g4};
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const int e = 3 * r + c;
            const double f = w * lx[r] * ly[c];
            L->re[e] = fma(f, kre, L->re[e]);
            if constexpr (KERNEL == BEM_HELMHOLTZ) L->im[e] = fma(f, kim, L->im[e]);
          }
      }
    }
  }
  for (int e = 0; e < 9; ++e) {
    L->re[e] = wave_sum(L->re[e]) * pg.scale;
    if constexpr (KERNEL == BEM_HELMHOLTZ) L->im[e] = wave_sum(L->im[e]) * pg.scale;
  }
}

template <int KERNEL>
__device__ __forceinline__ void store9(const P1Args &a, int64_t k, const Acc9<KERNEL> &L) {
  bool finite = true;
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    const int64_t dst = 9 * k + 3 * L.pr[e / 3] + L.pc[e % 3];
    if constexpr (KERNEL == BEM_LAPLACE) {
      static_cast<double *>(a.out)[dst] = L.re[e];
      finite = finite && isfinite(L.re[e]);
    } else {
      static_cast<double2 *>(a.out)[dst] = make_double2(L.re[e], L.im[e]);
      finite = finite && isfinite(L.re[e]) && isfinite(L.im[e]);
    }
  }
  if (!finite) atomicOr(a.flags, FLAG_NONFINITE);
}

// G lanes per regular pair, as in the kernel of arbitrary entries.
template <int KERNEL, int LAYER, int G, int XC>
__global__ __launch_bounds__(kThreads) void k_p1_pairs(const P1Args a) {
  constexpr int E = kThreads / G;  // pairs of a workgroup
  __shared__ int list[E];
  __shared__ int count;
  const int tid = threadIdx.x, sub = tid % G;
  if (tid == 0) count = 0;
  __syncthreads();
  const int64_t e = (int64_t)blockIdx.x * E + tid / G;
  int i = -1, j = -1;
  bool regular = false;
  if (e < a.n) {
    i = a.rows[e], j = a.cols[e];
    if (i < 0 || i >= a.nt || j < 0 || j >= a.nt) {
      atomicOr(a.flags, FLAG_EINVAL);
    } else {
      const int cls = shared_vertex_count(a.tri[3 * (int64_t)i], a.tri[3 * (int64_t)i + 1],
                                          a.tri[3 * (int64_t)i + 2], a.tri[3 * (int64_t)j],
                                          a.tri[3 * (int64_t)j + 1], a.tri[3 * (int64_t)j + 2]);
      regular = cls == 0;
      if (cls && sub == 0) list[atomicAdd(&count, 1)] = tid / G;
    }
  }
  if (regular) {  // the lanes of a pair together
    Acc9<KERNEL> L;
    p1_regular<KERNEL, LAYER, XC>(a, i, j, sub, G, &L);
#pragma unroll
    for (int o = G / 2; o >= 1; o /= 2)
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        L.re[k] += __shfl_xor(L.re[k], o, kWave);
        if constexpr (KERNEL == BEM_HELMHOLTZ) L.im[k] += __shfl_xor(L.im[k], o, kWave);
      }
    if (sub == 0) store9<KERNEL>(a, e, L);
  }
  __syncthreads();
  const int ns = count, wave = tid / kWave, lane = tid & (kWave - 1);
  for (int it = wave; it < ns; it += kThreads / kWave) {
    const int64_t ee = (int64_t)blockIdx.x * E + list[it];
    const int i = a.rows[ee], j = a.cols[ee];
    const int cls = shared_vertex_count(a.tri[3 * (int64_t)i], a.tri[3 * (int64_t)i + 1],
                                        a.tri[3 * (int64_t)i + 2], a.tri[3 * (int64_t)j],
                                        a.tri[3 * (int64_t)j + 1], a.tri[3 * (int64_t)j + 2]);
    Acc9<KERNEL> L;
    p1_singular<KERNEL, LAYER>(a, i, j, cls, &L);
    if (lane == 0) store9<KERNEL>(a, ee, L);
  }
}

// out[v + nrv w] = sum over (ta, ka) around row vertex v and (tb, kb) around
// column vertex w of local[(ta ntc + tb) 9 + 3 ka + kb], in list order.
template <bool CPLX>
__global__ __launch_bounds__(kThreads) void k_p1_gather(const P1GatherArgs a) {
  const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (e >= (int64_t)a.nrv * a.ncv) return;
  const int v = (int)(e % a.nrv), w = (int)(e / a.nrv);
  const int r0 = a.rs_ptr[v], r1 = a.rs_ptr[v + 1], c0 = a.cs_ptr[w], c1 = a.cs_ptr[w + 1];
  if (r0 < 0 || r0 > r1 || r1 > a.rs_len || c0 < 0 || c0 > c1 || c1 > a.cs_len) {
    atomicOr(a.flags, FLAG_EINVAL);
    return;
  }
  // a row triangle's products kQ at a time: their index and value loads are
  // issued together (one by one, each waits for the last: 32 us for a block of
  // 200 x 200 vertices)
  constexpr int kQ = 8;
  double re = 0.0, im = 0.0;
  for (int p = r0; p < r1; ++p) {
    const int ta = a.rs_tri[p], ka = a.rs_loc[p];
    const bool row = ta >= 0 && ta < a.ntr && ka >= 0 && ka <= 2;
    for (int q = c0; q < c1; q += kQ) {
      int64_t at[kQ];
      bool ok[kQ];
#pragma unroll
      for (int u = 0; u < kQ; ++u) {
        const bool in = q + u < c1;
        const int tb = in ? a.cs_tri[q + u] : 0, kb = in ? a.cs_loc[q + u] : 0;
        ok[u] = row && tb >= 0 && tb < a.ntc && kb >= 0 && kb <= 2;
        if (in && !ok[u]) atomicOr(a.flags, FLAG_EINVAL);
        ok[u] = ok[u] && in;
        at[u] = ((int64_t)ta * a.ntc + tb) * 9 + 3 * ka + kb;
      }
      double vr[kQ], vi[kQ];
#pragma unroll
      for (int u = 0; u < kQ; ++u) {
        const double *v = static_cast<const double *>(a.local) + (CPLX ? 2 : 1) * at[u];
        vr[u] = ok[u] ? v[0] : 0.0;
        vi[u] = CPLX && ok[u] ? v[1] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < kQ; ++u)
        if (ok[u]) re += vr[u], im += vi[u];
    }
  }
  if (CPLX) static_cast<double2 *>(a.out)[e] = make_double2(re, im);
  else static_cast<double *>(a.out)[e] = re;
}

// lanes per pair: see the kernel of arbitrary entries; 4 lanes and one, order 4,
// Laplace / Helmholtz: 200000 pairs 66 / 142 and 69 / 157 us, 440000 120 / 288 and
// 105 / 262.  One lane also leaves long lists all of a launch's 2^32 threads.
template <int KERNEL, int LAYER>
void launch_p1_kl(const P1Args &a, hipStream_t s) {
  const dim3 block(kThreads);
  auto grid = [&](int G) { return dim3((unsigned)((a.n * G + kThreads - 1) / kThreads)); };
  if (a.n < (1 << 15)) hipLaunchKernelGGL((k_p1_pairs<KERNEL, LAYER, 16, 1>), grid(16), block, 0, s, a);
  else if (a.n < (1 << 18)) hipLaunchKernelGGL((k_p1_pairs<KERNEL, LAYER, 4, 4>), grid(4), block, 0, s, a);
  else hipLaunchKernelGGL((k_p1_pairs<KERNEL, LAYER, 1, 4>), grid(1), block, 0, s, a);
}

}  // namespace

hipError_t launch_p1_pairs(int kernel, int layer, const P1Args &a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  if (kernel == BEM_LAPLACE) {
    if (layer == BEM_SLP) launch_p1_kl<BEM_LAPLACE, BEM_SLP>(a, s);
    else launch_p1_kl<BEM_LAPLACE, BEM_DLP>(a, s);
  } else {
    if (layer == BEM_SLP) launch_p1_kl<BEM_HELMHOLTZ, BEM_SLP>(a, s);
    else launch_p1_kl<BEM_HELMHOLTZ, BEM_DLP>(a, s);
  }
  return hipGetLastError();
}

hipError_t launch_p1_gather(bool cplx, const P1GatherArgs &a, hipStream_t s) {
  const int64_t n = (int64_t)a.nrv * a.ncv;
  if (n == 0) return hipSuccess;
  const dim3 grid((unsigned)((n + kThreads - 1) / kThreads)), block(kThreads);
  if (cplx) hipLaunchKernelGGL(k_p1_gather<true>, grid, block, 0, s, a);
  else hipLaunchKernelGGL(k_p1_gather<false>, grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace bem
