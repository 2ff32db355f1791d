// HIP kernels for gfx950 (CDNA4, wave64): per-triangle geometry and the
// evaluation of arbitrary entry lists.  The block kernel is in bem_blocks.hip.
#include <hip/hip_runtime.h>

#include <mutex>

#include "bem_device.h"

namespace bem {
namespace {

using namespace dev;

// ---------------------------------------------------------------- geometry
__global__ void k_geometry(const double *v, int32_t nv, const int32_t *tri, int32_t nt,
                           double *geo, int64_t ldg, unsigned *flags) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nt) return;
  const int a = tri[3 * (int64_t)i], b = tri[3 * (int64_t)i + 1], c = tri[3 * (int64_t)i + 2];
  double out[GEO_NF];
  for (int f = 0; f < GEO_NF; ++f) out[f] = 0.0;
  if (a < 0 || a >= nv || b < 0 || b >= nv || c < 0 || c >= nv) {
    atomicOr(flags, FLAG_EINVAL);
  } else {
    double p0[3], p1[3], p2[3];
    for (int k = 0; k < 3; ++k) {
      p0[k] = v[3 * (int64_t)a + k];
      p1[k] = v[3 * (int64_t)b + k];
      p2[k] = v[3 * (int64_t)c + k];
    }
    double e1[3], e2[3];
    for (int k = 0; k < 3; ++k) e1[k] = p1[k] - p0[k], e2[k] = p2[k] - p1[k];
    const double n0 = e1[1] * e2[2] - e1[2] * e2[1];
    const double n1 = e1[2] * e2[0] - e1[0] * e2[2];
    const double n2 = e1[0] * e2[1] - e1[1] * e2[0];
    const double sg = sqrt(n0 * n0 + n1 * n1 + n2 * n2);
    if (!(sg > 0.0) || !isfinite(sg)) atomicOr(flags, FLAG_EINVAL);
    for (int k = 0; k < 3; ++k) {
      out[G_V0X + k] = p0[k];
      out[G_E1X + k] = e1[k];
      out[G_E2X + k] = e2[k];
      out[G_LOX + k] = fmin(p0[k], fmin(p1[k], p2[k]));
      out[G_HIX + k] = fmax(p0[k], fmax(p1[k], p2[k]));
    }
    double g0 = 0.0, g1 = 0.0, g2 = 0.0;  // three times the vertices relative to the centroid
    for (int k = 0; k < 3; ++k) {
      const double p = 2.0 * e1[k] + e2[k], q = e1[k] - e2[k], r = e1[k] + 2.0 * e2[k];
      g0 = fma(p, p, g0), g1 = fma(q, q, g1), g2 = fma(r, r, g2);
    }
    out[G_R2] = fmax(g0, fmax(g1, g2)) * (1.0 / 9.0);
    out[G_SG] = sg;
    out[G_NX] = n0 / sg;
    out[G_NY] = n1 / sg;
    out[G_NZ] = n2 / sg;
  }
  for (int f = 0; f < GEO_NF; ++f) geo[f * ldg + i] = out[f];
}

// ---------------------------------------------------------------- entries
// Arbitrary (i, j) list: G lanes per regular entry (FP64, points formed on the
// fly; each lane takes every G-th chunk of XC x-points, their parts are added
// by lane shuffles); singular entries are listed and done by whole waves.  The
// mixed form stores the FP64 values rounded to FP32.
template <int KERNEL, int LAYER, bool MIXED, int G, int XC>
__global__ __launch_bounds__(kThreads) void k_entries(const EntryArgs a) {
  constexpr int E = kThreads / G;  // entries of a workgroup
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
  // the lanes of an entry take this branch together
  if (regular) {
    Acc<KERNEL> v = regular_pair_fp64<KERNEL, LAYER, XC>(a.geo, a.ldg, a.rule, a.nq, a.kappa, i, j,
                                                         sub, G);
#pragma unroll
    for (int o = G / 2; o >= 1; o /= 2) {
      v.re += __shfl_xor(v.re, o, kWave);
      if constexpr (KERNEL == BEM_HELMHOLTZ) v.im += __shfl_xor(v.im, o, kWave);
    }
    if (sub == 0) store_as<KERNEL, MIXED>(a.out, e, v, a.flags);
  }
  __syncthreads();
  const int ns = count, wave = tid / kWave, lane = tid & (kWave - 1);
  for (int it = wave; it < ns; it += kThreads / kWave) {
    const int64_t ee = (int64_t)blockIdx.x * E + list[it];
    const int si = a.rows[ee], sj = a.cols[ee];
    const int cls = shared_vertex_count(a.tri[3 * (int64_t)si], a.tri[3 * (int64_t)si + 1],
                                        a.tri[3 * (int64_t)si + 2], a.tri[3 * (int64_t)sj],
                                        a.tri[3 * (int64_t)sj + 1], a.tri[3 * (int64_t)sj + 2]);
    PairGeo g;
    if (pair_geometry(a.v, a.tri, a.nv, a.geo, a.ldg, si, sj, cls, a.flags, &g)) {
      const Acc<KERNEL> v = ss_pair_wave<KERNEL, LAYER>(g, a.ss, cls, a.kappa);
      if (lane == 0) store_as<KERNEL, MIXED>(a.out, ee, v, a.flags);
    }
  }
}

// Lanes per entry: one lane's chain over all nq^2 point pairs takes tens of
// microseconds, so a short list spreads each entry over 16 lanes (one x-point
// each in turn) and a middling one over 4; from kEntriesWide entries on, one
// lane each fills the GPU (two waves per SIMD) without the shared setup.
constexpr int64_t kEntriesShort = 1 << 15, kEntriesWide = 1 << 17;

template <int KERNEL, int LAYER, bool MIXED>
void launch_entries_klm(const EntryArgs &a, hipStream_t s) {
  const dim3 block(kThreads);
  auto grid = [&](int G) { return dim3((unsigned)((a.n * G + kThreads - 1) / kThreads)); };
  if (a.n < kEntriesShort) hipLaunchKernelGGL((k_entries<KERNEL, LAYER, MIXED, 16, 1>), grid(16), block, 0, s, a);
  else if (a.n < kEntriesWide) hipLaunchKernelGGL((k_entries<KERNEL, LAYER, MIXED, 4, 4>), grid(4), block, 0, s, a);
  else hipLaunchKernelGGL((k_entries<KERNEL, LAYER, MIXED, 1, 4>), grid(1), block, 0, s, a);
}

template <int KERNEL, int LAYER>
void launch_entries_kl(bool mixed, const EntryArgs &a, hipStream_t s) {
  if (mixed) launch_entries_klm<KERNEL, LAYER, true>(a, s);
  else launch_entries_klm<KERNEL, LAYER, false>(a, s);
}

// Fixed triangle-geometry scratch of the allocation-free near-field entry
// point: GEO_NF fields of up to BEM_NOALLOC_MAX_TRI triangles (leading
// dimension BEM_NOALLOC_MAX_TRI), one copy per GPU, held until the process
// ends.  Host code never passes this name to a kernel: it is a host-side
// stand-in; the device address comes from hipGetSymbolAddress.
static __device__ __align__(256) double scratch[GEO_NF * (size_t)BEM_NOALLOC_MAX_TRI];

}  // namespace

hipError_t noalloc_scratch(int device, double **ptr) {
  // the array's address on each device, looked up once with that device
  // current (the caller makes it current) and kept
  static std::mutex mu;
  static double *addr[64] = {};
  if (device < 0 || device >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[device]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[device] = static_cast<double *>(p);
  }
  *ptr = addr[device];
  return hipSuccess;
}

hipError_t launch_geometry(const bem_mesh &m, double *geo, int64_t ldg, unsigned *flags,
                           hipStream_t s) {
  if (m.nt == 0) return hipSuccess;
  hipLaunchKernelGGL(k_geometry, dim3((m.nt + 255) / 256), dim3(256), 0, s, m.v, m.nv, m.tri,
                     m.nt, geo, ldg, flags);
  return hipGetLastError();
}

hipError_t launch_entries(int kernel, int layer, bool mixed, const EntryArgs &a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  if (kernel == BEM_LAPLACE) {
    if (layer == BEM_SLP) launch_entries_kl<BEM_LAPLACE, BEM_SLP>(mixed, a, s);
    else launch_entries_kl<BEM_LAPLACE, BEM_DLP>(mixed, a, s);
  } else {
    if (layer == BEM_SLP) launch_entries_kl<BEM_HELMHOLTZ, BEM_SLP>(mixed, a, s);
    else launch_entries_kl<BEM_HELMHOLTZ, BEM_DLP>(mixed, a, s);
  }
  return hipGetLastError();
}

}  // namespace bem
