// Block assembly kernels (gfx950, wave64).  One sub-tile (up to 64 x 64
// entries of one block G[t x s]; up to 128 x 96 for a plain coupling block)
// is processed by one workgroup: regular pairs one entry per lane, the rest
// (singular pairs; near-singular pairs in the mixed form) grouped by class in
// LDS and done one pair per lane in FP64.
//   k_blocks      a block's sub-tiles dealt to gridDim.y workgroups, each
//                 looping over its share (one layer, or the single and the
//                 double layer in one pass);
//   k_persistent  a fixed grid of workgroups popping sub-tiles of many
//                 blocks (of many meshes) from a cost-sorted global queue.
// Both call the same sub-tile code, so their results are bitwise equal.
// Instantiated per kernel and precision by the bem_blocks_*.hip files.
#pragma once

#include <hip/hip_runtime.h>

#include "bem_block_core.h"
#include "bem_block_launch.h"

namespace bem {
namespace {

using namespace blk;

// The thread's index, read through an empty asm statement: values derived
// from it (lane, strides of the staging loops, LDS offsets) are then formed
// where they are used instead of being hoisted to the kernel's entry and
// held, or spilled, across the sub-tile loops (the block kernels drop 30 to
// 50 registers and their scratch spills this way).
__device__ __forceinline__ int thread_id() {
  int t = __builtin_amdgcn_workitem_id_x();
  asm volatile("" : "+v"(t));
  return t;
}

struct BlockHdr {
  int64_t rp0, cp0, nr, nc, off;
  int64_t moff;       // transposed copy (coupling of a single layer), -1: none
  bool diag;          // its own mirror (moff == off): a block on the diagonal,
                      // only its entries with row >= column are evaluated
  bool brief;         // block_is_brief
  double cx, cy, cz;  // block-local origin: first vertex of the first row triangle
};

// Validates block b of a block list; false (and the flag) if its ranges or
// output slot are invalid.  Uniform across the workgroup.
__device__ __forceinline__ bool block_header(const BlockArgs &a, int b, BlockHdr *h) {
  const int64_t rp0 = a.row_ptr[b], rp1 = a.row_ptr[b + 1];
  const int64_t cp0 = a.col_ptr[b], cp1 = a.col_ptr[b + 1];
  const int64_t off = a.out_off[b];
  bool ok = rp0 >= 0 && rp0 <= rp1 && rp1 <= a.row_len && cp0 >= 0 && cp0 <= cp1 &&
            cp1 <= a.col_len && off >= 0 && off <= a.out_len;
  const int64_t nr = rp1 - rp0, nc = cp1 - cp0;
  ok = ok && (nr == 0 || nc <= (a.out_len - off) / nr);
  int i0 = 0;
  if (ok && nr > 0 && nc > 0) {
    i0 = a.row_idx[rp0];
    ok = i0 >= 0 && i0 < a.nt;
  }
  if (!ok) {
    if (thread_id() == 0) atomicOr(a.flags, FLAG_EINVAL);
    return false;
  }
  h->rp0 = rp0;
  h->cp0 = cp0;
  h->nr = nr;
  h->nc = nc;
  h->off = off;
  h->moff = a.mirror_off ? a.mirror_off[b] : -1;
  h->diag = h->moff >= 0 && h->moff == off && nr == nc;
  if (h->moff >= 0 && nr > 0 && !h->diag &&
      (h->moff == off || h->moff > a.out_len || nc > (a.out_len - h->moff) / nr)) {
    if (thread_id() == 0) atomicOr(a.flags, FLAG_EINVAL);  // onto itself, or does not fit
    h->moff = -1;
  }
  if (nr > 0 && nc > 0) {
    h->cx = a.geo[G_V0X * a.ldg + i0];
    h->cy = a.geo[G_V0Y * a.ldg + i0];
    h->cz = a.geo[G_V0Z * a.ldg + i0];
  }
  return true;
}

// Whether block h may take its Helmholtz phases relative to the centroids'
// distance: is_brief for every triangle of its rows and columns.  A property of the block
// alone, so that its entries do not depend on the kernel or the sub-tiles that
// compute them, and one for all its entries: with a decision per entry, waves
// that held both kinds ran both sums (0.64x on a coarse mesh).  Uniform; starts
// and ends with a barrier.
template <int KERNEL>
__device__ bool block_is_brief(const BlockArgs &a, const Lds &l, const BlockHdr &h) {
  if constexpr (KERNEL == BEM_LAPLACE) {
    return false;
  } else {
    const int tid = thread_id();
    __syncthreads();
    if (tid == 0) *l.bad = 0;
    __syncthreads();
    for (int64_t k = tid; k < h.nr + h.nc; k += kThreads) {
      const int id = k < h.nr ? a.row_idx[h.rp0 + k] : a.col_idx[h.cp0 + (k - h.nr)];
      if (!is_brief(a, id)) *l.bad = 1;
    }
    __syncthreads();
    const bool brief = *l.bad == 0;
    __syncthreads();
    return brief;
  }
}

// The quadrature rule into LDS.
__device__ __forceinline__ void load_rule(const BlockArgs &a, const Lds &l) {
  const int nqp = a.nq_pad, nq = a.nq;
  for (int k = thread_id(); k < nq; k += kThreads) {
    l.rule[k] = a.rule[k];
    l.rule[nqp + k] = a.rule[nq + k];
    l.rule[2 * nqp + k] = a.rule[2 * nq + k];
  }
}

// Phase A of a sub-tile (rows r0 .. r0 + tr, columns c0 .. c0 + tc): reset
// the counters, then triangle ids (validated), vertex ids, row geometry in
// block-local coordinates and column normals (and boxes in the mixed form).
// Starts with a barrier (the previous sub-tile is done with the LDS) and ends
// with one; false (uniformly, flag raised) if a triangle id is invalid.
template <bool MIXED>
__device__ bool stage_tile(const BlockArgs &a, const Lds &l, const BlockHdr &h, int64_t r0,
                           int64_t c0, int tr, int tc) {
  const int tid = thread_id(), TR = a.tr, TC = a.tc;
  const int64_t L = a.ldg;
  const double cx = h.cx, cy = h.cy, cz = h.cz;
  __syncthreads();
  if (tid < 16) l.ccount[tid] = 0, l.cursor[tid] = 0;
  if (tid == 0) *l.count = 0, *l.bad = 0, *l.rcount = 0;
  __syncthreads();
  for (int k = tid; k < tr + tc; k += kThreads) {
    const bool isrow = k < tr;
    const int id = isrow ? a.row_idx[h.rp0 + r0 + k] : a.col_idx[h.cp0 + c0 + (k - tr)];
    if (id < 0 || id >= a.nt) {
      *l.bad = 1;
      continue;
    }
    double e1[3], e2[3];
    for (int m = 0; m < 3; ++m) {
      e1[m] = a.geo[(G_E1X + m) * L + id];
      e2[m] = a.geo[(G_E2X + m) * L + id];
    }
    if (isrow) {
      l.rid[k] = id;
      for (int m = 0; m < 3; ++m) l.rv[m * TR + k] = a.tri[3 * (int64_t)id + m];
      l.rg[(R_V + 0) * TR + k] = 2.0 * (a.geo[G_V0X * L + id] - cx);
      l.rg[(R_V + 1) * TR + k] = 2.0 * (a.geo[G_V0Y * L + id] - cy);
      l.rg[(R_V + 2) * TR + k] = 2.0 * (a.geo[G_V0Z * L + id] - cz);
      double aa = 0.0, ab = 0.0, bb = 0.0;
      for (int m = 0; m < 3; ++m) {
        const double A = 2.0 * fma(2.0, e1[m], e2[m]), B = 4.0 * e2[m];
        l.rg[(R_A + m) * TR + k] = A;
        l.rg[(R_B + m) * TR + k] = B;
        aa = fma(A, A, aa), ab = fma(A, B, ab), bb = fma(B, B, bb);
      }
      l.rg[R_SG * TR + k] = a.geo[G_SG * L + id];
      l.rg[R_C1 * TR + k] = 0.5 * ab;
      l.rg[R_K0 * TR + k] = 0.25 * aa;
      l.rg[R_A22 * TR + k] = 0.25 * bb;
      if (l.rn) {
        l.rn[k] = a.geo[G_NX * L + id];
        l.rn[TR + k] = a.geo[G_NY * L + id];
        l.rn[2 * TR + k] = a.geo[G_NZ * L + id];
      }
      if constexpr (MIXED)
        for (int m = 0; m < 6; ++m) l.rb[m * TR + k] = a.geo[(G_LOX + m) * L + id];
    } else {
      const int cl = k - tr;
      l.cid[cl] = id;
      for (int m = 0; m < 3; ++m) l.cv[m * TC + cl] = a.tri[3 * (int64_t)id + m];
      double yn = 0.0;
      for (int m = 0; m < 3; ++m) {
        const double c = m == 0 ? cx : m == 1 ? cy : cz;
        const double n = a.geo[(G_NX + m) * L + id], y = 2.0 * (a.geo[(G_V0X + m) * L + id] - c);
        l.cn[m * TC + cl] = n;
        l.cc[m * TC + cl] = fma(2.0 / 3.0, fma(2.0, e1[m], e2[m]), y);
        if constexpr (MIXED) l.cg[m * TC + cl] = y;
        yn = fma(y, n, yn);
      }
      l.cn[3 * TC + cl] = yn;
      if constexpr (MIXED)
        for (int m = 0; m < 6; ++m) l.cb[m * TC + cl] = a.geo[(G_LOX + m) * L + id];
    }
  }
  __syncthreads();
  if (*l.bad) {
    if (tid == 0) atomicOr(a.flags, FLAG_EINVAL);
    return false;
  }
  return true;
}

// The sub-tile's column triangles [kColumnFields][TC] into l.ys: 2 (v0 - c),
// 2 e1, 2 e2 and sqrt(g).
__device__ __forceinline__ void stage_triangles(const BlockArgs &a, const Lds &l, const BlockHdr &h, int tc) {
  for (int k = thread_id(); k < tc * kColumnFields; k += kThreads) {
    const int cl = k % tc, m = k / tc, id = l.cid[cl];
    const double x = a.geo[(m < 9 ? G_V0X + m : G_SG) * a.ldg + id];
    l.ys[m * a.tc + cl] = m == 9 ? x : 2.0 * (m == 0 ? x - h.cx : m == 1 ? x - h.cy : m == 2 ? x - h.cz : x);
  }
}

// Phase B: what the regular sums keep of the columns, then a barrier.
// Rules with kernels of their own: the column points of the rule in l.rule.  General rules: the triangles, and 4 |y - c|^2 of every point.
template <int RULE, bool MIXED>
__device__ void stage_columns(const BlockArgs &a, const Lds &l, const BlockHdr &h, int tc) {
  const int TC = a.tc, nqp = a.nq_pad;
  const int64_t L = a.ldg;
  const double cx = h.cx, cy = h.cy, cz = h.cz;
  // relative to the triangle's first vertex, resp. centroid
  constexpr bool LOCAL = MIXED || RULE >= kRule4;
  constexpr double s0 = RULE >= kRule4 ? 2.0 / 3.0 : 0.0, t0 = 0.5 * s0;
  if constexpr (RULE >= kRule4) stage_triangles(a, l, h, tc);
  for (int k = thread_id(); k < tc * a.nq; k += kThreads) {
    const int cl = k % tc, q = k / tc;
    const int id = l.cid[cl];
    const double s = l.rule[q] - s0, t = l.rule[nqp + q] - t0;
    const double P0 = 2.0 * fma(s, a.geo[G_E1X * L + id], fma(t, a.geo[G_E2X * L + id], LOCAL ? 0.0 : a.geo[G_V0X * L + id] - cx));
    const double P1 = 2.0 * fma(s, a.geo[G_E1Y * L + id], fma(t, a.geo[G_E2Y * L + id], LOCAL ? 0.0 : a.geo[G_V0Y * L + id] - cy));
    const double P2 = 2.0 * fma(s, a.geo[G_E1Z * L + id], fma(t, a.geo[G_E2Z * L + id], LOCAL ? 0.0 : a.geo[G_V0Z * L + id] - cz));
    if constexpr (RULE >= kRule4) {
      typedef typename std::conditional<MIXED, float, double>::type T;
      reinterpret_cast<T *>(l.ys + kColumnFields * TC)[q * TC + cl] = (T)fma(P0, P0, fma(P1, P1, P2 * P2));
    } else {
      const double W = l.rule[2 * nqp + q] * a.geo[G_SG * L + id];
      if constexpr (!MIXED) {
        double2 *y = reinterpret_cast<double2 *>(l.ys) + 2 * ((int64_t)q * TC + cl);
        y[0] = make_double2(P0, P1);
        y[1] = make_double2(P2, W);
      } else {
        float4 *y = reinterpret_cast<float4 *>(l.ys) + ((int64_t)q * TC + cl);
        *y = make_float4((float)P0, (float)P1, (float)P2, (float)W);
      }
    }
  }
  __syncthreads();
}

// Phase D: the listed pairs (front of l.list, *l.count of them) grouped by
// class (identical, edge, vertex, near-singular) into l.sorted, each group
// padded to a multiple of 64 with kNoPair so that every wave-sized chunk
// holds one class.  Expects a barrier after the listing; ends with one
// unless nothing is listed.
struct Groups {
  int seg[4];  // start of the group of class c
  int total;   // padded length
};

__device__ __forceinline__ Groups group_listed(const Lds &l) {
  const int tid = thread_id();
  const int ns = *l.count;
  Groups g;
  const int n3 = (l.ccount[3] + 63) & ~63, n2 = (l.ccount[2] + 63) & ~63,
            n1 = (l.ccount[1] + 63) & ~63, n0 = (l.ccount[0] + 63) & ~63;
  g.seg[0] = n3 + n2 + n1;
  g.seg[1] = n3 + n2;
  g.seg[2] = n3;
  g.seg[3] = 0;
  g.total = n3 + n2 + n1 + n0;
  if (ns == 0) return g;  // uniform
  for (int k = tid; k < g.total; k += kThreads) l.sorted[k] = kNoPair;
  __syncthreads();
  for (int k = tid; k < ns; k += kThreads) {
    const uint16_t code = l.list[k];
    const int cls = (code >> 12) & 3;
    l.sorted[g.seg[cls] + atomicAdd(&l.cursor[cls], 1)] = code;
  }
  __syncthreads();
  return g;
}

// Phase E for one wave-sized chunk of the grouped list (chunk start pos):
// one pair per lane in FP64.
template <int KERNEL, int LAYER, bool MIXED>
__device__ __forceinline__ void singular_chunk(const BlockArgs &a, const Lds &l,
                                               const BlockHdr &h, int64_t r0, int64_t c0,
                                               const Groups &gr, int pos) {
  const int lane = thread_id() & (kWave - 1);
  const int cls = pos < gr.seg[2] ? CLS_IDENTICAL
                  : pos < gr.seg[1] ? CLS_EDGE
                  : pos < gr.seg[0] ? CLS_VERTEX : kNearSingular;
  const uint16_t code = l.sorted[pos + lane];
  const bool active = code != kNoPair;
  const bool swapped = active && (code & kSwapped);
  const int rl = code & 63, cl = (code >> 6) & 63;
  // a swapped code is the mirror block's entry: the pair (j, i) to (c, r)
  const int64_t dst = swapped ? h.moff + (c0 + cl) + h.nc * (r0 + rl)
                              : h.off + (r0 + rl) + h.nr * (c0 + cl);
  const int64_t mdst = h.moff >= 0 && !swapped && cls != CLS_EDGE
                           ? h.moff + (c0 + cl) + h.nc * (r0 + rl) : -1;
  if (cls == kNearSingular) {
    if (active) {
      const Acc<KERNEL> v = regular_pair_fp64<KERNEL, LAYER>(a.geo, a.ldg, a.rule, a.nq, a.kappa,
                                                             l.rid[rl], l.cid[cl]);
      store_as<KERNEL, MIXED>(a.out, dst, v, a.flags);
      if (mdst >= 0) store_as<KERNEL, MIXED>(a.out, mdst, v, a.flags);
    }
    return;
  }
  PairGeo g;
  bool have = false;
  if (active)
    have = pair_geometry(a.v, a.tri, a.nv, a.geo, a.ldg, swapped ? l.cid[cl] : l.rid[rl],
                         swapped ? l.rid[rl] : l.cid[cl], cls, a.flags, &g);
  if (!have) {  // idle lane: harmless finite geometry, result discarded
    for (int c = 0; c < 3; ++c)
      g.E1i[c] = c == 0, g.E2i[c] = c == 1, g.E1j[c] = -(c == 2), g.E2j[c] = 0, g.n[c] = 0;
    g.scale = 0.0;
  }
  Acc<KERNEL> v;
  ss_pair_lane<KERNEL, LAYER>(g, a.ss, cls, a.kappa, LAYER == BEM_SLP ? &v : nullptr,
                              LAYER == BEM_SLP ? nullptr : &v);
  if (have) {
    store_as<KERNEL, MIXED>(a.out, dst, v, a.flags);
    if (mdst >= 0) store_as<KERNEL, MIXED>(a.out, mdst, v, a.flags);
  }
}

// Phase E of the one-pass form (both layers, in FP64): the pair (i, j) of a
// listed code in both layers and, if the block has a mirror, the transposed
// pair (j, i): an edge pair evaluated as (j, i) (that rule is not symmetric);
// else its single layer copied and its double layer summed over the same
// directions (vertex pairs) or point pairs (near-singular pairs).  The class is uniform
// across the chunk.
template <int KERNEL, bool MIXED>
__device__ __forceinline__ void singular_chunk_both(const BlockArgs &a, const Lds &l,
                                                    const BlockHdr &h, int64_t r0, int64_t c0,
                                                    const Groups &gr, int pos) {
  const int lane = thread_id() & (kWave - 1);
  const int cls = pos < gr.seg[2] ? CLS_IDENTICAL
                  : pos < gr.seg[1] ? CLS_EDGE
                  : pos < gr.seg[0] ? CLS_VERTEX : kNearSingular;
  const uint16_t code = l.sorted[pos + lane];
  const bool active = code != kNoPair;
  const int rl = code & 63, cl = (code >> 6) & 63;
  const int64_t dst = h.off + (r0 + rl) + h.nr * (c0 + cl);
  const int64_t mdst = h.moff + (c0 + cl) + h.nc * (r0 + rl);
  if (cls == kNearSingular) {  // mixed form: a regular pair summed in FP64
    if (!active) return;
    const int i = l.rid[rl], j = l.cid[cl];
    Acc<KERNEL> vs, vd, md;
    regular_pair_both_fp64<KERNEL>(a.geo, a.ldg, a.rule, a.nq, a.kappa, i, j, &vs, &vd, &md);
    store_as<KERNEL, MIXED>(a.out, dst, vs, a.flags);
    store_as<KERNEL, MIXED>(a.out2, dst, vd, a.flags);
    if (h.moff >= 0) {
      store_as<KERNEL, MIXED>(a.out, mdst, vs, a.flags);
      store_as<KERNEL, MIXED>(a.out2, mdst, md, a.flags);
    }
    return;
  }
  auto idle = [](PairGeo *g) {  // harmless finite geometry, result discarded
    for (int c = 0; c < 3; ++c)
      g->E1i[c] = c == 0, g->E2i[c] = c == 1, g->E1j[c] = -(c == 2), g->E2j[c] = 0, g->n[c] = 0;
    g->scale = 0.0;
  };
  PairGeo g;
  bool have = false;
  if (active)
    have = pair_geometry(a.v, a.tri, a.nv, a.geo, a.ldg, l.rid[rl], l.cid[cl], cls, a.flags, &g);
  if (!have) idle(&g);
  // a vertex pair's directions serve (j, i) too: its rule is symmetric (the
  // class and the mirror are uniform across the wave)
  const bool mirror = h.moff >= 0 && !(h.diag && cls == CLS_IDENTICAL);
  Acc<KERNEL> vs, vd, md;
  if (cls == CLS_VERTEX && mirror) {
    double ni[3] = {0.0, 0.0, 0.0};
    if (have)
      for (int c = 0; c < 3; ++c) ni[c] = l.rn[c * a.tr + rl];
    ss_pair_lane<KERNEL, kSS, true>(g, a.ss, cls, a.kappa, &vs, &vd, &md, ni);
  } else {
    ss_pair_lane<KERNEL, kSS>(g, a.ss, cls, a.kappa, &vs, &vd);
  }
  if (have) {
    store_as<KERNEL, MIXED>(a.out, dst, vs, a.flags);
    store_as<KERNEL, MIXED>(a.out2, dst, vd, a.flags);
  }
  // uniform: no mirror, or an identical pair of a diagonal block (its own
  // transpose, already written)
  if (!mirror) return;
  Acc<KERNEL> ms = vs;
  if (cls == CLS_EDGE) {
    have = false;
    if (active)
      have = pair_geometry(a.v, a.tri, a.nv, a.geo, a.ldg, l.cid[cl], l.rid[rl], cls, a.flags, &g);
    if (!have) idle(&g);
    ss_pair_lane<KERNEL, kSS>(g, a.ss, cls, a.kappa, &ms, &md);
  }
  if (have) {
    store_as<KERNEL, MIXED>(a.out, mdst, ms, a.flags);
    store_as<KERNEL, MIXED>(a.out2, mdst, md, a.flags);
  }
}

// Near-singular pair of the mixed form: bounding boxes closer than ratio * the
// larger box diagonal.  row(m), col(m): component m of the boxes (lower corner,
// upper corner).
template <class R, class C>
__device__ __forceinline__ bool near_pair(double ratio, R &&row, C &&col) {
  double gap2 = 0.0, di = 0.0, dj = 0.0;
  for (int m = 0; m < 3; ++m) {
    const double rlo = row(m), rhi = row(3 + m), clo = col(m), chi = col(3 + m);
    const double g = fmax(0.0, fmax(clo - rhi, rlo - chi));
    gap2 = fma(g, g, gap2);
    di = fma(rhi - rlo, rhi - rlo, di);
    dj = fma(chi - clo, chi - clo, dj);
  }
  return gap2 < ratio * ratio * fmax(di, dj);
}

// Whether entry (rl, cl) of the staged sub-tile goes to the FP64 pass:
// a common vertex (cls > 0), or in the mixed form a near-singular pair.
template <bool MIXED>
__device__ __forceinline__ bool fp64_pair(const Lds &l, int TR, int TC, int rl, int cl,
                                          double ratio, int *cls_out) {
  const int cls = shared_vertex_count(l.rv[rl], l.rv[TR + rl], l.rv[2 * TR + rl], l.cv[cl],
                                      l.cv[TC + cl], l.cv[2 * TC + cl]);
  *cls_out = cls;
  bool fp64 = cls != 0;
  if constexpr (MIXED) {
    if (!fp64 && ratio > 0.0)
      fp64 = near_pair(ratio, [&](int m) { return l.rb[m * TR + rl]; }, [&](int m) { return l.cb[m * TC + cl]; });
  }
  return fp64;
}

// Pairs that the full sub-tile around the staged one, a.wide columns, lists in a
// mirrored list (edge-adjacent ones twice).  Uniform; with barriers.
template <bool MIXED>
__device__ int full_count(const BlockArgs &a, const Lds &l, const BlockHdr &h, int64_t r0, int64_t c0, int tr) {
  const int tid = thread_id(), TR = a.tr;
  const int64_t w0 = c0 - c0 % a.wide;
  const int wc = (int)min((int64_t)a.wide, h.nc - w0);
  __syncthreads();
  if (tid == 0) *l.bad = 0;
  __syncthreads();
  for (int e = tid; e < tr * wc; e += kThreads) {
    const int rl = e % tr;
    const int64_t c = w0 + e / tr;
    if (h.diag && r0 + rl < c) continue;
    const int id = a.col_idx[h.cp0 + c];
    if (id < 0 || id >= a.nt) continue;  // reported by its own sub-tile
    const int32_t *v = a.tri + 3 * (int64_t)id;
    const int cls = shared_vertex_count(l.rv[rl], l.rv[TR + rl], l.rv[2 * TR + rl], v[0], v[1], v[2]);
    int n = cls == 0 ? 0 : cls == CLS_EDGE ? 2 : 1;
    if constexpr (MIXED) {
      if (cls == 0 && a.near_ratio > 0.0)
        n = near_pair(a.near_ratio, [&](int m) { return l.rb[m * TR + rl]; },
                      [&](int m) { return a.geo[(G_LOX + m) * a.ldg + id]; });
    }
    if (n) atomicAdd(l.bad, n);
  }
  __syncthreads();
  return *l.bad;
}

// Entry e of the lower triangle (row >= column) of an n x n tile, columns
// in turn: column c holds rows c .. n - 1 and starts at S(c) = c n - c (c -
// 1) / 2; the FP32 estimate of c is corrected to the exact one.
__device__ __forceinline__ void lower_entry(int e, int n, int *rl, int *cl) {
  const float b = 2.0f * n + 1.0f;
  int c = (int)((b - sqrtf(fmaxf(b * b - 8.0f * e, 0.0f))) * 0.5f);
  c = max(0, min(c, n - 1));
  while (c > 0 && c * n - c * (c - 1) / 2 > e) --c;
  while (c + 1 < n && (c + 1) * n - (c + 1) * c / 2 <= e) ++c;
  *cl = c;
  *rl = c + (e - (c * n - c * (c - 1) / 2));
}

// The factors left out of the sums: 1/(4 pi), and 1/2 of the doubled normal
// distance for the double layers.
template <int KERNEL>
__device__ __forceinline__ void scale_sums(Sums<KERNEL> *o) {
  const double fs = kInv4Pi, fd = 0.5 * kInv4Pi;
  o->s.re *= fs;
  o->d.re *= fd;
  o->m.re *= fd;
  if constexpr (KERNEL == BEM_HELMHOLTZ) o->s.im *= fs, o->d.im *= fd, o->m.im *= fd;
}

// One sub-tile: rows r0 .. r0 + TR, columns c0 .. c0 + TC of the block
// (LAYER = kBoth: the single layer to a.out and the double layer to a.out2).
// After staging, the pairs of the FP64 pass are listed and grouped by class;
// then every wave takes work from one counter -- first the FP64 chunks
// (heaviest), then the regular entries 64 at a time in column-major order
// (lanes of a chunk share a column, so column points are broadcast reads)
// -- until both are done, so the FP64 work is spread over the waves instead
// of ending the sub-tile.  Returns early (uniformly) if a triangle id is
// invalid.
template <int KERNEL, int LAYER, int RULE, bool MIXED>
__device__ void subtile(const BlockArgs &a, const Lds &l, const BlockHdr &h, int64_t r0,
                        int64_t c0, int coupling) {
  const int tid = thread_id(), lane = tid & (kWave - 1);
  const int TR = a.tr, TC = a.tc;
  const int64_t nr = h.nr, off = h.off;
  const double ratio = a.near_ratio;
  const int tr = (int)min((int64_t)TR, h.nr - r0), tc = (int)min((int64_t)TC, h.nc - c0);
  // a diagonal block evaluates its entries with row >= column only (the
  // rest are their transposes): a sub-tile wholly above the diagonal is
  // skipped, a square one on it enumerates its lower triangle
  if (h.diag && r0 + tr - 1 < c0) return;  // uniform
  const bool lower = h.diag && r0 == c0 && tr == tc;
  const bool upper_skip = h.diag && !lower;
  if (!stage_tile<MIXED>(a, l, h, r0, c0, tr, tc)) return;
  stage_columns<RULE, MIXED>(a, l, h, tc);
  // phase C: list the pairs of the FP64 pass
  for (int e = tid; e < tr * tc; e += kThreads) {
    const int rl = e % tr, cl = e / tr;
    if (h.diag && r0 + rl < c0 + cl) continue;
    int cls;
    if (!fp64_pair<MIXED>(l, TR, TC, rl, cl, ratio, &cls)) continue;
    if (coupling && cls) {
      atomicOr(a.flags, FLAG_EINVAL);
    } else {
      // an edge-adjacent pair of a mirrored block is listed twice: the
      // mirror's entry is evaluated as (j, i)
      const bool twice = LAYER != kBoth && h.moff >= 0 && cls == CLS_EDGE;
      const uint16_t code = (uint16_t)(rl | (cl << 6) | (cls << 12));
      const int n = twice ? 2 : 1;
      const int slot = atomicAdd(l.count, n);
      if (slot + n <= a.slots) {  // else the sub-tile fails below
        l.list[slot] = code;
        if (twice) l.list[slot + 1] = code | kSwapped;
      }
      atomicAdd(&l.ccount[cls], n);
    }
  }
  __syncthreads();
  // more listed pairs than entries (a mirrored list): too many if those of the
  // full sub-tile are
  if (*l.count > TR * TC && (*l.count > a.slots || full_count<MIXED>(a, l, h, r0, c0, tr) > TR * a.wide)) {
    if (tid == 0) atomicOr(a.flags, FLAG_LIST);  // uniform
    return;
  }
  const Groups gr = group_listed(l);
  const int nreg = lower ? tr * (tr + 1) / 2 : tr * tc;
  const int nsc = gr.total / kWave, nrc = (nreg + kWave - 1) / kWave;
  for (;;) {
    int c = 0;
    if (lane == 0) c = atomicAdd(l.rcount, 1);
    c = __builtin_amdgcn_readfirstlane(c);  // uniform: the chunk's class too, its tables by scalar loads
    if (c >= nsc + nrc) break;
    if (c < nsc) {
      if constexpr (LAYER == kBoth) {
        singular_chunk_both<KERNEL, MIXED>(a, l, h, r0, c0, gr, c * kWave);
      } else {
        singular_chunk<KERNEL, LAYER, MIXED>(a, l, h, r0, c0, gr, c * kWave);
      }
      continue;
    }
    const int e = (c - nsc) * kWave + lane;
    if (e >= nreg) continue;
    int rl, cl;
    if (lower) {
      lower_entry(e, tr, &rl, &cl);
    } else {
      rl = e % tr, cl = e / tr;
      if (upper_skip && r0 + rl < c0 + cl) continue;
    }
    int cls;
    if (fp64_pair<MIXED>(l, TR, TC, rl, cl, ratio, &cls)) continue;
    Sums<KERNEL> o;
    regular_sums<KERNEL, LAYER, RULE, MIXED>(l, TR, TC, a.nq, rl, cl, a.sums, a.rule, a.kappa, h.brief, &o);
    scale_sums(&o);
    const int64_t dst = off + (r0 + rl) + nr * (c0 + cl);
    const int64_t mdst = h.moff + (c0 + cl) + h.nc * (r0 + rl);
    store_as<KERNEL, MIXED>(a.out, dst, LAYER == BEM_DLP ? o.d : o.s, a.flags);
    if constexpr (LAYER == kBoth) store_as<KERNEL, MIXED>(a.out2, dst, o.d, a.flags);
    if (h.moff >= 0) {
      store_as<KERNEL, MIXED>(a.out, mdst, LAYER == BEM_DLP ? o.d : o.s, a.flags);
      if constexpr (LAYER == kBoth) store_as<KERNEL, MIXED>(a.out2, mdst, o.m, a.flags);
    }
  }
}

// Sums of a regular entry of the learned form: order Q on both triangles.
template <int KERNEL, int LAYER, int Q>
__device__ __forceinline__ void learned_sums(const Lds &l, int TR, int TC, int rl, int cl,
                                             const OrderRules &o, double kappa, bool brief,
                                             Sums<KERNEL> *v) {
  const EntryGeo g = entry_geo<LAYER, false>(l, TR, TC, rl, cl);
  const PointsOfRule pts{l.ys + cl, TC, (uniform_ptr)o.rule[Q], Q * Q};
  if (KERNEL == BEM_HELMHOLTZ && brief) duffy_sums<KERNEL, LAYER, Q, true, double>(g, o.duffy[Q], kappa, pts, v);
  else duffy_sums<KERNEL, LAYER, Q, false, double>(g, o.duffy[Q], kappa, pts, v);
}

// Sub-tile of the learned form (plain FP64): every regular entry takes the
// Duffy/Gauss order of the order map (2 .. q_max); the entries are grouped by
// order (each group padded to a multiple of 64, one order per wave-sized
// chunk).  Singular pairs as in the plain kernel.  The column points are formed
// from the staged triangle as they are used (six operations for the q^2 point
// pairs of each): staged per order they kept the orders apart by barriers, the
// waves idle for 39 % of the time (8192 triangles, Helmholtz, orders 2 to 5: 2.65
// -> 2.34 ms; 4608, order 6: 2.53 -> 2.01; Laplace, 8192: 0.77 -> 0.71).
template <int KERNEL, int LAYER>
__device__ void subtile_learned(const BlockArgs &a, const OrderRules &o, const Lds &l,
                                const BlockHdr &h, int64_t r0, int64_t c0) {
  const int tid = thread_id(), lane = tid & (kWave - 1);
  const int TR = a.tr, TC = a.tc;
  const int64_t nr = h.nr, off = h.off;
  const int tr = (int)min((int64_t)TR, h.nr - r0), tc = (int)min((int64_t)TC, h.nc - c0);
  const int cap = a.slots;
  if (!stage_tile<false>(a, l, h, r0, c0, tr, tc)) return;
  stage_triangles(a, l, h, tc);
  // classify: singular pairs to the front of the list, regular ones (with
  // their order) to the back
  for (int e = tid; e < tr * tc; e += kThreads) {
    const int rl = e % tr, cl = e / tr;
    const int cls = shared_vertex_count(l.rv[rl], l.rv[TR + rl], l.rv[2 * TR + rl], l.cv[cl],
                                        l.cv[TC + cl], l.cv[2 * TC + cl]);
    if (cls) {
      l.list[atomicAdd(l.count, 1)] = (uint16_t)(rl | (cl << 6) | (cls << 12));
      atomicAdd(&l.ccount[cls], 1);
      continue;
    }
    const int q = o.orders[off + (r0 + rl) + nr * (c0 + cl)];
    if (q < 2 || q > o.q_max) {
      atomicOr(a.flags, FLAG_EINVAL);
      continue;
    }
    l.list[cap - 1 - atomicAdd(l.rcount, 1)] = (uint16_t)(rl | (cl << 6) | (q << 12));
    atomicAdd(&l.ccount[8 + q], 1);
  }
  __syncthreads();
  // the singular pairs grouped by class at the front of sorted[], then the
  // regular ones by descending order (each group padded to a multiple of 64):
  // roughly by descending cost of a chunk
  const Groups gr = group_listed(l);
  const int nreg = *l.rcount;
  int seg[7];
  int total = gr.total;
  for (int q = o.q_max; q >= 2; --q) {
    seg[q] = total;
    total += (l.ccount[8 + q] + 63) & ~63;
  }
  for (int k = gr.total + tid; k < total; k += kThreads) l.sorted[k] = kNoPair;
  __syncthreads();
  for (int k = tid; k < nreg; k += kThreads) {
    const uint16_t code = l.list[cap - 1 - k];
    const int q = code >> 12;
    l.sorted[seg[q] + atomicAdd(&l.cursor[8 + q], 1)] = code;
  }
  __syncthreads();
  // the waves take chunks from one counter (zeroed by stage_tile)
  const int nsc = gr.total / kWave;
  for (;;) {
    int c = 0;
    if (lane == 0) c = atomicAdd(&l.cursor[15], 1);
    c = __builtin_amdgcn_readfirstlane(c);
    if (c >= total / kWave) break;
    if (c < nsc) {
      singular_chunk<KERNEL, LAYER, false>(a, l, h, r0, c0, gr, c * kWave);
      continue;
    }
    const uint16_t code = l.sorted[c * kWave + lane];
    const int q = __builtin_amdgcn_readfirstlane(code) >> 12;  // lane 0 of a chunk has a pair
    if (code == kNoPair) continue;
    const int rl = code & 63, cl = (code >> 6) & 63;
    Sums<KERNEL> v;
    switch (q) {
      case 2: learned_sums<KERNEL, LAYER, 2>(l, TR, TC, rl, cl, o, a.kappa, h.brief, &v); break;
      case 3: learned_sums<KERNEL, LAYER, 3>(l, TR, TC, rl, cl, o, a.kappa, h.brief, &v); break;
      case 4: learned_sums<KERNEL, LAYER, 4>(l, TR, TC, rl, cl, o, a.kappa, h.brief, &v); break;
      case 5: learned_sums<KERNEL, LAYER, 5>(l, TR, TC, rl, cl, o, a.kappa, h.brief, &v); break;
      default: learned_sums<KERNEL, LAYER, 6>(l, TR, TC, rl, cl, o, a.kappa, h.brief, &v);
    }
    scale_sums(&v);
    store_as<KERNEL, false>(a.out, off + (r0 + rl) + nr * (c0 + cl), LAYER == BEM_DLP ? v.d : v.s,
                            a.flags);
  }
}

template <int KERNEL, int LAYER>
__global__ __launch_bounds__(kThreads, 2) void k_blocks_learned(const BlockArgs a,
                                                                const OrderRules o) {
  extern __shared__ __align__(16) double lds_raw[];  // 16-byte aligned: ds_read_b128 of points
  BlockHdr h;
  if (!block_header(a, blockIdx.x, &h) || h.nr == 0 || h.nc == 0) return;
  const Lds l = carve<false>(lds_raw, a);
  h.brief = block_is_brief<KERNEL>(a, l, h);
  unsigned turn = blockIdx.y;  // as k_blocks
  for (int64_t r0 = 0; r0 < h.nr; r0 += a.tr)
    for (int64_t c0 = 0; c0 < h.nc; c0 += a.tc) {
      if (turn == 0) subtile_learned<KERNEL, LAYER>(a, o, l, h, r0, c0);
      turn = turn == 0 ? gridDim.y - 1 : turn - 1;
    }
}

template <int KERNEL, int LAYER, int RULE, bool MIXED>
__global__ __launch_bounds__(kThreads, 2) void k_blocks(const BlockArgs a, const int coupling) {
  extern __shared__ __align__(16) double lds_raw[];  // 16-byte aligned: ds_read_b128 of points
  BlockHdr h;
  if (!block_header(a, blockIdx.x, &h) || h.nr == 0 || h.nc == 0) return;
  const Lds l = carve<MIXED>(lds_raw, a, LAYER == kBoth);
  h.brief = RULE < kSeven && block_is_brief<KERNEL>(a, l, h);
  load_rule(a, l);
  // the block's sub-tiles, dealt to gridDim.y workgroups
  unsigned turn = blockIdx.y;
  for (int64_t r0 = 0; r0 < h.nr; r0 += a.tr)
    for (int64_t c0 = 0; c0 < h.nc; c0 += a.tc) {
      if (turn == 0) subtile<KERNEL, LAYER, RULE, MIXED>(a, l, h, r0, c0, coupling);
      turn = turn == 0 ? gridDim.y - 1 : turn - 1;
    }
}

// Persistent form: every workgroup pops work items (batch, block, r0, c0) --
// one sub-tile, or the whole block when r0 = c0 = -1 -- from a queue sorted by
// decreasing cost until it is empty; every batch shares the operator's kernel,
// precision and rules and has its own mesh, blocks, layer (single, double or
// both in one pass), sub-tile shape and output.
// Copy of a read-only struct at a wave-uniform address by scalar loads.
template <class T>
__device__ __forceinline__ T uniform_copy(const T *p) {
  static_assert(sizeof(T) % 4 == 0, "dword-sized struct");
  typedef const uint32_t __attribute__((address_space(4))) *cword_t;
  T v;
  const cword_t src = (cword_t)p;
  uint32_t *dst = reinterpret_cast<uint32_t *>(&v);
#pragma unroll
  for (int k = 0; k < (int)(sizeof(T) / 4); ++k) dst[k] = src[k];
  return v;
}

// One work item of batch entry d.x in the layer LAYER: the argument and
// header checks, the LDS layout of the entry's sub-tile shape (the rule,
// shared by every entry, loaded again where that layout moves it; no wave
// reads the LDS between the queue's barriers and the first barrier of the
// sub-tile's staging), then the sub-tile or the whole block.  Each layer has
// its own copy, so that nothing but the queue state is live across the
// choice of layer.
template <int KERNEL, int LAYER, int RULE, bool MIXED>
__device__ __forceinline__ void persistent_item(const BlockArgs *__restrict__ batches, int4 d, int cp,
                                                double *lds_raw, int *carved) {
  // the entry's arguments are read where used (scalar loads from read-only
  // memory, which the compiler may repeat instead of holding or spilling
  // them across the sub-tile loops)
  const BlockArgs &a = batches[d.x];
  if (d.y < 0 || d.y >= a.nblocks) {
    if (thread_id() == 0) atomicOr(a.flags, FLAG_EINVAL);
    return;
  }
  BlockHdr h;
  if (!block_header(a, d.y, &h) || h.nr == 0 || h.nc == 0) return;
  const bool whole = d.z == -1 && d.w == -1;
  if (!whole && (d.z >= h.nr || d.w >= h.nc || d.z < 0 || d.w < 0)) {
    if (thread_id() == 0) atomicOr(a.flags, FLAG_EINVAL);
    return;
  }
  const Lds l = carve<MIXED>(lds_raw, a, LAYER == kBoth);
  const int shape = a.tr | (a.tc << 10);
  if (shape != *carved) {
    load_rule(a, l);
    *carved = shape;
  }
  h.brief = KERNEL == BEM_HELMHOLTZ && RULE < kSeven &&
            (a.brief ? a.brief[d.y] != 0 : block_is_brief<KERNEL>(a, l, h));
  if (whole) {  // the whole block, sub-tile by sub-tile
    for (int64_t r0 = 0; r0 < h.nr; r0 += a.tr)
      for (int64_t c0 = 0; c0 < h.nc; c0 += a.tc) subtile<KERNEL, LAYER, RULE, MIXED>(a, l, h, r0, c0, cp);
  } else {
    subtile<KERNEL, LAYER, RULE, MIXED>(a, l, h, d.z, d.w, cp);
  }
}

template <int KERNEL, int RULE, bool MIXED>
__global__ __launch_bounds__(kThreads, 2) void k_persistent(const BlockArgs *__restrict__ batches,
                                                            const int32_t *mode,
                                                            const int4 *tiles, int32_t ntiles,
                                                            int32_t nbatch, int32_t *counter) {
  extern __shared__ __align__(16) double lds_raw[];  // 16-byte aligned: ds_read_b128 of points
  __shared__ int s_tile;
  // the queue and the batch arguments are read-only here: their loads have
  // wave-uniform addresses and are scalar, as the per-block kernel's
  // argument loads
  typedef const int32_t __attribute__((address_space(4))) *cint_t;
  int carved = -1;  // sub-tile shape whose LDS layout holds the rule, -1: none yet
  for (;;) {
    __syncthreads();  // everyone has read s_tile and left the previous tile
    if (thread_id() == 0) s_tile = atomicAdd(counter, 1);
    __syncthreads();
    const int t = __builtin_amdgcn_readfirstlane(s_tile);
    if (t >= ntiles) break;  // the counter only grows: every workgroup exits
    const int4 d = uniform_copy(tiles + t);
    const int md = d.x >= 0 && d.x < nbatch ? ((cint_t)mode)[d.x] : -1;
    const int cp = md & 1, layer = md >> 1;
    if (layer == BEM_SLP) {
      persistent_item<KERNEL, BEM_SLP, RULE, MIXED>(batches, d, cp, lds_raw, &carved);
    } else if (layer == BEM_DLP) {
      persistent_item<KERNEL, BEM_DLP, RULE, MIXED>(batches, d, cp, lds_raw, &carved);
    } else if (layer == kBoth) {
      persistent_item<KERNEL, kBoth, RULE, MIXED>(batches, d, cp, lds_raw, &carved);
    } else if (thread_id() == 0) {  // batch index or mode out of range
      atomicOr(batches->flags, FLAG_EINVAL);
    }
  }
}

template <int KERNEL, bool MIXED, int RULE>
hipError_t launch_rule(int layer, bool coupling, const BlockArgs &a, size_t lds, hipStream_t s) {
  const dim3 grid(a.nblocks, a.split), block(kThreads);
  const int cp = coupling ? 1 : 0;
  if (layer == BEM_SLP) hipLaunchKernelGGL((k_blocks<KERNEL, BEM_SLP, RULE, MIXED>), grid, block, lds, s, a, cp);
  else if (layer == BEM_DLP) hipLaunchKernelGGL((k_blocks<KERNEL, BEM_DLP, RULE, MIXED>), grid, block, lds, s, a, cp);
  else hipLaunchKernelGGL((k_blocks<KERNEL, kBoth, RULE, MIXED>), grid, block, lds, s, a, cp);
  return hipGetLastError();
}

// f(integral constant of the rule variant).  Helmholtz takes chunks of 4 in
// place of 8 and 9, whose sines and cosines would not fit the registers.
template <int KERNEL, class F>
hipError_t with_rule(int rule, F &&f) {
  constexpr bool HELM = KERNEL == BEM_HELMHOLTZ;
  switch (rule) {
    case 2: return f(std::integral_constant<int, 2>{});
    case 3: return f(std::integral_constant<int, 3>{});
    case 4: return f(std::integral_constant<int, 4>{});
    case 5: return f(std::integral_constant<int, 5>{});
    case 6: return f(std::integral_constant<int, 6>{});
    case kSeven: return f(std::integral_constant<int, kSeven>{});
    case kRule7: return f(std::integral_constant<int, kRule7>{});
    case kRule8: return f(std::integral_constant<int, HELM ? kRule4 : kRule8>{});
    case kRule9: return f(std::integral_constant<int, HELM ? kRule4 : kRule9>{});
    case kRule4: return f(std::integral_constant<int, kRule4>{});
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

template <int KERNEL, bool MIXED>
hipError_t BlockLaunch<KERNEL, MIXED>::blocks(int layer, int rule, bool coupling, const BlockArgs &a,
                                              size_t lds, hipStream_t s) {
  return with_rule<KERNEL>(rule, [&](auto r) {
    return launch_rule<KERNEL, MIXED, decltype(r)::value>(layer, coupling, a, lds, s);
  });
}

template <int KERNEL, bool MIXED>
hipError_t PersistentLaunch<KERNEL, MIXED>::run(int rule, const PersistentArgs &p, size_t lds,
                                                hipStream_t s) {
  return with_rule<KERNEL>(rule, [&](auto r) {
    hipLaunchKernelGGL((k_persistent<KERNEL, decltype(r)::value, MIXED>), dim3(p.grid), dim3(kThreads),
                       lds, s, p.batches, p.mode, p.tiles, p.ntiles, p.nbatch, p.counter);
    return hipGetLastError();
  });
}

template <int KERNEL>
hipError_t LearnedLaunch<KERNEL>::run(int layer, const BlockArgs &a, const OrderRules &o, size_t lds,
                                      hipStream_t s) {
  const dim3 grid(a.nblocks, a.split), block(kThreads);
  if (layer == BEM_SLP) hipLaunchKernelGGL((k_blocks_learned<KERNEL, BEM_SLP>), grid, block, lds, s, a, o);
  else hipLaunchKernelGGL((k_blocks_learned<KERNEL, BEM_DLP>), grid, block, lds, s, a, o);
  return hipGetLastError();
}

}  // namespace bem
