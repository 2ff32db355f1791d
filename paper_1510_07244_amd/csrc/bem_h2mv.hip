// Matrix-vector kernels of the H^2 matrix (Sec. 2.3-2.4: near-field blocks,
// nested cluster bases, coupling matrices) and the vector operations of the
// iterative solvers that use it (Sec. 4: conjugate gradients for the Laplace
// single layer; the Brakhage-Werner system for Helmholtz).
//
// The product is a handful of grouped, gathered small matrix-vector products
// (forward transformation of the column basis, coupling, backward
// transformation of the row basis, near field).  Each reads its matrices
// once, so it is bound by HBM bandwidth, not arithmetic: the kernels read
// every matrix column-wise with 64 consecutive lanes on 64 consecutive rows
// (one 512-byte line per wave and column), and the waves of a workgroup work
// on different blocks without barriers between them.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "bem_device.h"

namespace bem {
namespace {

using namespace dev;

constexpr int kMaxVec = 512;  // longest output and input of one group / block

// v of lane k, k uniform across the wave (two scalar reads of the halves)
__device__ __forceinline__ double read_lane(double v, int k) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), k);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), k);
  return __hiloint2double(hi, lo);
}

template <bool CPLX>
struct Num;
template <>
struct Num<false> {
  double v;
  __device__ static Num zero() { Num r; r.v = 0.0; return r; }
  __device__ void fma(const Num &m, const Num &x) { v = ::fma(m.v, x.v, v); }
  __device__ static Num load(const double *p, int64_t k) { Num r; r.v = p[k]; return r; }
  __device__ void add_to(double *p, int64_t k) const { p[k] += v; }
  __device__ void add(const Num &o) { v += o.v; }
  __device__ Num xor_lane(int o) const { Num r; r.v = __shfl_xor(v, o, kWave); return r; }
  // the value of lane k (k uniform across the wave)
  __device__ Num lane(int k) const { Num r; r.v = read_lane(v, k); return r; }
};
template <>
struct Num<true> {
  double re, im;
  __device__ static Num zero() { Num r; r.re = r.im = 0.0; return r; }
  __device__ void fma(const Num &m, const Num &x) {
    re = ::fma(m.re, x.re, re);
    re = ::fma(-m.im, x.im, re);
    im = ::fma(m.re, x.im, im);
    im = ::fma(m.im, x.re, im);
  }
  __device__ static Num load(const double *p, int64_t k) {
    Num r;
    r.re = p[2 * k];
    r.im = p[2 * k + 1];
    return r;
  }
  __device__ void add_to(double *p, int64_t k) const {
    p[2 * k] += re;
    p[2 * k + 1] += im;
  }
  __device__ void add(const Num &o) { re += o.re, im += o.im; }
  __device__ Num xor_lane(int o) const {
    Num r;
    r.re = __shfl_xor(re, o, kWave);
    r.im = __shfl_xor(im, o, kWave);
    return r;
  }
  __device__ Num lane(int k) const {
    Num r;
    r.re = read_lane(re, k);
    r.im = read_lane(im, k);
    return r;
  }
};

// Group g: y[out_idx[out_ptr[g] ..]] += sum_{b in group g} op(A_b) x[in_idx[in_ptr[b] ..]],
// op(A) = A (TRANS false; A is m_out x n_in) or A^T (TRANS true; A is
// n_in x m_out), column-major with the row count as leading dimension.
//
// A level of the nested basis has few groups of small blocks (13 to 182 for
// 8192 triangles), so a launch is bound by the latency of one workgroup's
// chain (offsets -> indices -> inputs, matrix entries) and by how many
// workgroups share the matrices, not by bandwidth.  A group's outputs are
// therefore spread over gridDim.y workgroups, which need nothing from each
// other: 64 output rows each (TRANS false, one line of 512 bytes per column) or one panel of kPanel
// output columns (TRANS true).  Within a
// workgroup the waves take the group's work in turn -- panels of kPanel input
// columns, resp. 64-row pieces of the blocks -- each issuing a panel's loads
// before it uses them, and their partial sums are added in wave order: every
// sum runs in a fixed order, so results are reproducible bit for bit.
// One product of the 8192-triangle single layer (224 MB, graph replay, every
// matrix from HBM): 230 us with one workgroup per group, its rows in two passes
// and six shuffles per column -> 157 us; the transposed levels 10 .. 13 -> 6 ..
// 9 us each, the coupling 56 -> 43 us (3.2 TB/s).  Tried: pieces of 32 rows or
// of 128 with 16-byte loads (coupling 62 and 53 us), eight waves (164 us),
// the blocks' list entries loaded 64 at a time (159 us).
constexpr int kGemvThreads = 1024;
constexpr int kGemvWaves = kGemvThreads / kWave;
template <bool CPLX>
constexpr int kPanel = CPLX ? 8 : 16;

// element k of a list the kernel only reads, k uniform: a scalar load
__device__ __forceinline__ int64_t list_at(const int32_t *p, int64_t k) {
  return ((const int32_t __attribute__((address_space(4))) *)p)[k];
}
__device__ __forceinline__ int64_t list_at(const int64_t *p, int64_t k) {
  return ((const int64_t __attribute__((address_space(4))) *)p)[k];
}

struct GemvGroup {
  int64_t o0, b0, b1;
  int m;
};

// Offsets of group g; false (and the flag) if they are invalid.  Uniform.
__device__ __forceinline__ bool gemv_group(const GemvArgs &a, int g, GemvGroup *r) {
  const int64_t o0 = list_at(a.out_ptr, g), o1 = list_at(a.out_ptr, g + 1);
  r->o0 = o0;
  r->b0 = list_at(a.grp_ptr, g), r->b1 = list_at(a.grp_ptr, g + 1);
  if (o0 >= 0 && o0 <= o1 && o1 <= a.out_len && o1 - o0 <= kMaxVec && r->b0 >= 0 &&
      r->b0 <= r->b1 && r->b1 <= a.nblocks) {
    r->m = (int)(o1 - o0);
    return true;
  }
  if (threadIdx.x == 0) atomicOr(a.flags, FLAG_EINVAL);
  return false;
}

// Input range and matrix of block b with m output rows / columns; false (and
// the flag) if they are invalid.  Uniform in a wave.
struct GemvBlock {
  int64_t i0, off;
  int n;
};
__device__ __forceinline__ bool gemv_block(const GemvArgs &a, int64_t b, int m, int lane,
                                           GemvBlock *r) {
  const int64_t i0 = list_at(a.in_ptr, b), i1 = list_at(a.in_ptr, b + 1), off = list_at(a.a_off, b);
  const int64_t n = i1 - i0;
  r->i0 = i0, r->off = off;
  if (i0 >= 0 && i0 <= i1 && i1 <= a.in_len && n <= kMaxVec && off >= 0 && off <= a.a_len &&
      (m == 0 || n <= (a.a_len - off) / m)) {
    r->n = (int)n;
    return true;
  }
  if (lane == 0) atomicOr(a.flags, FLAG_EINVAL);
  return false;
}

template <bool CPLX>
__device__ __forceinline__ Num<CPLX> gemv_input(const GemvArgs &a, int64_t k, bool in) {
  Num<CPLX> v = Num<CPLX>::zero();
  if (in) {
    const int id = a.in_idx[k];
    if (id >= 0 && id < a.x_len) v = Num<CPLX>::load(static_cast<const double *>(a.x), id);
    else atomicOr(a.flags, FLAG_EINVAL);
  }
  return v;
}

// entry k of the matrix at the wave-uniform address base: scalar base and a
// 32-bit byte offset (m, n <= 512), half the address registers of 64-bit ones
template <bool CPLX>
__device__ __forceinline__ Num<CPLX> load_entry(const double *base, int k) {
  const uint32_t off = (uint32_t)k * (CPLX ? 16u : 8u);
  return Num<CPLX>::load(reinterpret_cast<const double *>(reinterpret_cast<const char *>(base) + off), 0);
}

template <bool CPLX>
__device__ __forceinline__ void gemv_add(const GemvArgs &a, int64_t k, const Num<CPLX> &v) {
  const int id = a.out_idx[k];
  if (id < 0 || id >= a.y_len) atomicOr(a.flags, FLAG_EINVAL);
  else v.add_to(static_cast<double *>(a.y), id);
}

// TRANS false: lane l takes output row l of a 64-row piece; the inputs of a
// panel are gathered one per lane, one panel ahead, and broadcast.
template <bool CPLX>
__global__ __launch_bounds__(kGemvThreads) void k_gemv(const GemvArgs a) {
  using T = Num<CPLX>;
  constexpr int P = kPanel<CPLX>;
  __shared__ T part[kGemvWaves][kWave];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  GemvGroup gr;
  if (!gemv_group(a, blockIdx.x, &gr)) return;
  const int m = gr.m;
  // (a group without outputs takes one turn, in which its blocks are checked)
  for (int r0 = blockIdx.y * kWave; r0 < max(m, 1); r0 += gridDim.y * kWave) {  // uniform
    const int row = r0 + lane;
    T acc = T::zero();
    int64_t task = 0;  // panels of the group's blocks so far
    for (int64_t b = gr.b0; b < gr.b1; ++b) {
      GemvBlock bl;
      const int64_t len = list_at(a.in_ptr, b + 1) - list_at(a.in_ptr, b);
      const int64_t np = (len + P - 1) / P;
      int64_t p = ((wave - task) % kGemvWaves + kGemvWaves) % kGemvWaves;  // first panel of block b
      task += np;
      if (p >= np || !gemv_block(a, b, m, lane, &bl)) continue;  // uniform in the wave
      T xl = gemv_input<CPLX>(a, bl.i0 + p * P + lane, lane < P && p * P + lane < bl.n);
      for (; p < np; p += kGemvWaves) {
        const int jn = min(P, bl.n - (int)p * P);
        const double *C = static_cast<const double *>(a.A) + (CPLX ? 2 : 1) * (bl.off + (int64_t)m * (p * P));
        T av[P];
#pragma unroll
        for (int u = 0; u < P; ++u) av[u] = row < m && u < jn ? load_entry<CPLX>(C, row + m * u) : T::zero();
        const int64_t pn = p + kGemvWaves;
        const T xn = gemv_input<CPLX>(a, bl.i0 + pn * P + lane, lane < P && pn * P + lane < bl.n);
#pragma unroll
        for (int u = 0; u < P; ++u) acc.fma(av[u], xl.lane(u));
        xl = xn;
      }
    }
    part[wave][lane] = acc;
    __syncthreads();
    if (tid < kWave && row < m) {
      T s = part[0][tid];
      for (int w = 1; w < kGemvWaves; ++w) s.add(part[w][tid]);
      gemv_add<CPLX>(a, gr.o0 + row, s);
    }
    __syncthreads();  // part is reused by the next rows
  }
}

// TRANS true: lane l takes input row l of a 64-row piece of a block and runs
// along the workgroup's panel of columns; the columns' sums over the lanes
// are formed by exchanging halves (after the first four, resp. three, steps
// a lane holds one column).
template <bool CPLX>
__global__ __launch_bounds__(kThreads, 4) void k_gemv_trans(const GemvArgs a) {
  using T = Num<CPLX>;
  constexpr int P = kPanel<CPLX>, W = kThreads / kWave;
  __shared__ T part[W][P];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const double *A = static_cast<const double *>(a.A);
  GemvGroup gr;
  if (!gemv_group(a, blockIdx.x, &gr)) return;
  const int m = gr.m;
  for (int j0 = blockIdx.y * P; j0 < m; j0 += gridDim.y * P) {  // uniform
    const int jn = min(P, m - j0);
    T s[P];
#pragma unroll
    for (int u = 0; u < P; ++u) s[u] = T::zero();
    int64_t task = 0;  // 64-row pieces of the group's blocks so far
    for (int64_t b = gr.b0; b < gr.b1; ++b) {
      GemvBlock bl;
      const int64_t len = list_at(a.in_ptr, b + 1) - list_at(a.in_ptr, b);
      const int64_t np = (len + kWave - 1) / kWave;
      int64_t p = ((wave - task) % W + W) % W;  // this wave's first piece of block b
      // (an empty block's range is checked too)
      task += max(np, (int64_t)0);
      if ((p >= np && len > 0) || !gemv_block(a, b, m, lane, &bl)) continue;  // uniform in the wave
      const double *C = A + (CPLX ? 2 : 1) * (bl.off + (int64_t)bl.n * j0);
      for (; p < np; p += W) {
        const int row = (int)p * kWave + lane;
        const bool in = row < bl.n;
        T av[P];
#pragma unroll
        for (int u = 0; u < P; ++u) av[u] = in && u < jn ? load_entry<CPLX>(C, row + bl.n * u) : T::zero();
        const T xi = gemv_input<CPLX>(a, bl.i0 + row, in);
#pragma unroll
        for (int u = 0; u < P; ++u) s[u].fma(av[u], xi);
      }
    }
    int mask = kWave / 2;
#pragma unroll
    for (int h = P / 2; h >= 1; h /= 2, mask /= 2) {
      const bool up = lane & mask;
#pragma unroll
      for (int u = 0; u < h; ++u) {
        T keep = up ? s[u + h] : s[u];
        keep.add((up ? s[u] : s[u + h]).xor_lane(mask));
        s[u] = keep;
      }
    }
    for (; mask >= 1; mask /= 2) s[0].add(s[0].xor_lane(mask));
    constexpr int kLanes = kWave / P;  // lanes that hold one column
    if (lane % kLanes == 0) part[wave][lane / kLanes] = s[0];
    __syncthreads();
    if (tid < jn) {
      T t = part[0][tid];
      for (int w = 1; w < W; ++w) t.add(part[w][tid]);
      gemv_add<CPLX>(a, gr.o0 + j0 + tid, t);
    }
    __syncthreads();  // part is reused by the next panel
  }
}

// ------------------------------------------------------------ vector ops
constexpr int kDotBlocks = 256;

// Partial sums of sum_i conj?(x_i) y_i: workgroup b takes the fixed strided
// set of indices b * 256 + t + 256 * 256 * r, reduced in a fixed order.
template <bool CPLX, bool CONJ>
__global__ __launch_bounds__(kThreads) void k_dot_part(int64_t n, const double *x, const double *y,
                                                       double *part) {
  __shared__ double sr[kThreads], si[kThreads];
  double re = 0.0, im = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads) {
    if (CPLX) {
      const double xr = x[2 * i], xi = CONJ ? -x[2 * i + 1] : x[2 * i + 1];
      const double yr = y[2 * i], yi = y[2 * i + 1];
      re = fma(xr, yr, re);
      re = fma(-xi, yi, re);
      im = fma(xr, yi, im);
      im = fma(xi, yr, im);
    } else {
      re = fma(x[i], y[i], re);
    }
  }
  sr[threadIdx.x] = re;
  si[threadIdx.x] = im;
  __syncthreads();
  for (int s = kThreads / 2; s >= 1; s >>= 1) {
    if ((int)threadIdx.x < s) {
      sr[threadIdx.x] += sr[threadIdx.x + s];
      si[threadIdx.x] += si[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = sr[0];
    part[2 * blockIdx.x + 1] = si[0];
  }
}

__global__ __launch_bounds__(kThreads) void k_dot_final(int nparts, const double *part,
                                                        double *out) {
  __shared__ double sr[kThreads], si[kThreads];
  double re = 0.0, im = 0.0;
  for (int k = threadIdx.x; k < nparts; k += kThreads) re += part[2 * k], im += part[2 * k + 1];
  sr[threadIdx.x] = re;
  si[threadIdx.x] = im;
  __syncthreads();
  for (int s = kThreads / 2; s >= 1; s >>= 1) {
    if ((int)threadIdx.x < s) {
      sr[threadIdx.x] += sr[threadIdx.x + s];
      si[threadIdx.x] += si[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = sr[0], out[1] = si[0];
}

// y = alpha x + beta y (complex alpha, beta; real vectors use the real parts)
template <bool CPLX>
__global__ __launch_bounds__(kThreads) void k_axpby(int64_t n, double ar, double ai,
                                                    const double *x, double br, double bi,
                                                    double *y) {
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads) {
    if (CPLX) {
      const double xr = x[2 * i], xi = x[2 * i + 1], yr = y[2 * i], yi = y[2 * i + 1];
      y[2 * i] = ar * xr - ai * xi + (br * yr - bi * yi);
      y[2 * i + 1] = ar * xi + ai * xr + (br * yi + bi * yr);
    } else {
      y[i] = ar * x[i] + br * y[i];
    }
  }
}

// y += c M x, M the Galerkin mass matrix of piecewise constants: diagonal,
// M_ii = |tau_i| = sqrt(g_i) / 2
template <bool CPLX>
__global__ __launch_bounds__(kThreads) void k_mass(int32_t nt, const double *geo, int64_t ldg,
                                                   double cr, double ci, const double *x,
                                                   double *y) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= nt) return;
  const double area = 0.5 * geo[G_SG * ldg + i];
  if (CPLX) {
    const double xr = x[2 * i], xi = x[2 * i + 1];
    y[2 * i] += area * (cr * xr - ci * xi);
    y[2 * i + 1] += area * (cr * xi + ci * xr);
  } else {
    y[i] += area * cr * x[i];
  }
}

// Conjugate-gradient updates with the step scalars in device memory (the
// layout of the state array is documented at bem_cg_step): the host reads
// them only to decide when to stop, not once per step.
__global__ __launch_bounds__(kThreads) void k_cg_xr(int64_t n, const double *st, const double *p,
                                                    const double *q, double *x, double *r) {
  const bool go = st[7] != 0.0 && st[2] != 0.0;
  const double alpha = go ? st[0] / st[2] : 0.0;
  const double one = 1.0;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads) {
    x[i] = alpha * p[i] + one * x[i];
    r[i] = -alpha * q[i] + one * r[i];
  }
}

__global__ __launch_bounds__(kThreads) void k_cg_p(int64_t n, const double *st, const double *r,
                                                   double *p) {
  if (!(st[7] != 0.0 && st[2] != 0.0)) return;  // uniform: stopped, p stays
  const double beta = st[4] / st[0];
  const double one = 1.0;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads)
    p[i] = one * r[i] + beta * p[i];
}

__global__ void k_cg_close(double *st) {
  if (st[7] == 0.0) return;
  if (st[2] == 0.0) {  // p.q = 0: breakdown, stop with the current iterate
    st[7] = 0.0;
    return;
  }
  st[0] = st[4];
  st[8] += 1.0;
  st[7] = st[0] > st[6] && st[8] < st[9] ? 1.0 : 0.0;
}

}  // namespace

hipError_t launch_cg_step(int64_t n, double *state, double *x, double *r, double *p,
                          const double *q, double *dot_part, hipStream_t s) {
  const dim3 grid((unsigned)std::min<int64_t>(std::max<int64_t>((n + kThreads - 1) / kThreads, 1), 4096)),
      block(kThreads);
  hipLaunchKernelGGL(k_cg_xr, grid, block, 0, s, n, state, p, q, x, r);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = launch_dot(false, false, n, r, r, dot_part, state + 4, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_cg_p, grid, block, 0, s, n, state, r, p);
  hipLaunchKernelGGL(k_cg_close, dim3(1), dim3(1), 0, s, state);
  return hipGetLastError();
}

hipError_t launch_gemv(bool cplx, bool trans, const GemvArgs &a, hipStream_t s) {
  if (a.ngroups == 0) return hipSuccess;
  // workgroups per group from the mean number of outputs (the lengths
  // themselves are device memory): pieces of rows of twice the mean (the
  // coupling's groups have 40 to 125 rows of mean 51), resp. panels of a quarter more than the mean; one
  // without work ends at once, one with more loops, so any number is correct
  const int64_t mean = std::max<int64_t>((a.out_len + a.ngroups - 1) / a.ngroups, 1);
  const int panel = cplx ? kPanel<true> : kPanel<false>;
  const int64_t want = trans ? (5 * mean / 4 + panel - 1) / panel : (2 * mean + kWave - 1) / kWave;
  const unsigned gy = (unsigned)std::min<int64_t>(std::max<int64_t>(want, 1), kMaxVec / panel);
  // a launch has 2^32 threads along the groups: more of them in turns
  constexpr int32_t kMost = 1 << 21;
  for (int32_t g0 = 0; g0 < a.ngroups; g0 += std::min(kMost, a.ngroups - g0)) {
    GemvArgs t = a;
    t.ngroups = std::min(kMost, a.ngroups - g0);
    t.grp_ptr += g0, t.out_ptr += g0;
    const dim3 grid((unsigned)t.ngroups, gy);
    if (cplx) {
      if (trans) hipLaunchKernelGGL(k_gemv_trans<true>, grid, dim3(kThreads), 0, s, t);
      else hipLaunchKernelGGL(k_gemv<true>, grid, dim3(kGemvThreads), 0, s, t);
    } else {
      if (trans) hipLaunchKernelGGL(k_gemv_trans<false>, grid, dim3(kThreads), 0, s, t);
      else hipLaunchKernelGGL(k_gemv<false>, grid, dim3(kGemvThreads), 0, s, t);
    }
  }
  return hipGetLastError();
}

size_t dot_scratch_doubles() { return 2 * kDotBlocks; }

hipError_t launch_dot(bool cplx, bool conj, int64_t n, const double *x, const double *y,
                      double *part, double *out, hipStream_t s) {
  const dim3 grid(kDotBlocks), block(kThreads);
  if (cplx) {
    if (conj) hipLaunchKernelGGL((k_dot_part<true, true>), grid, block, 0, s, n, x, y, part);
    else hipLaunchKernelGGL((k_dot_part<true, false>), grid, block, 0, s, n, x, y, part);
  } else {
    hipLaunchKernelGGL((k_dot_part<false, false>), grid, block, 0, s, n, x, y, part);
  }
  hipLaunchKernelGGL(k_dot_final, dim3(1), block, 0, s, kDotBlocks, part, out);
  return hipGetLastError();
}

hipError_t launch_axpby(bool cplx, int64_t n, double ar, double ai, const double *x, double br,
                        double bi, double *y, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const dim3 grid((unsigned)std::min<int64_t>((n + kThreads - 1) / kThreads, 4096)), block(kThreads);
  if (cplx) hipLaunchKernelGGL(k_axpby<true>, grid, block, 0, s, n, ar, ai, x, br, bi, y);
  else hipLaunchKernelGGL(k_axpby<false>, grid, block, 0, s, n, ar, ai, x, br, bi, y);
  return hipGetLastError();
}

hipError_t launch_mass(bool cplx, int32_t nt, const double *geo, int64_t ldg, double cr, double ci,
                       const double *x, double *y, hipStream_t s) {
  if (nt == 0) return hipSuccess;
  const dim3 grid((nt + kThreads - 1) / kThreads), block(kThreads);
  if (cplx) hipLaunchKernelGGL(k_mass<true>, grid, block, 0, s, nt, geo, ldg, cr, ci, x, y);
  else hipLaunchKernelGGL(k_mass<false>, grid, block, 0, s, nt, geo, ldg, cr, ci, x, y);
  return hipGetLastError();
}

}  // namespace bem
