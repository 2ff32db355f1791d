// Launch rules of the block assembly kernels: rule variants, sub-tile shapes
// and the dispatch to the instantiations (bem_blocks_*, bem_persistent_*,
// bem_learned_*.hip).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "bem_block_core.h"
#include "bem_block_launch.h"

namespace bem {
namespace {

__global__ void k_reset_counter(int32_t *counter) { *counter = 0; }

// The same, and one workgroup per block for its phase kind.
constexpr int kBeginThreads = 1024;
__global__ __launch_bounds__(kBeginThreads) void k_begin(int32_t *counter, const BlockArgs *batches,
                                                         int32_t nbatch) {
  constexpr int U = 4;  // triangles in flight
  const int tid = threadIdx.x;
  if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *counter = 0;
  for (int32_t k = blockIdx.y; k < nbatch; k += gridDim.y) {
    const BlockArgs &a = batches[k];
    if (!a.brief) continue;  // uniform
    for (int32_t b = blockIdx.x; b < a.nblocks; b += gridDim.x) {
      const int64_t rp0 = a.row_ptr[b], nr = a.row_ptr[b + 1] - rp0;
      const int64_t cp0 = a.col_ptr[b], nc = a.col_ptr[b + 1] - cp0;
      // ranges that block_header refuses: not read
      int bad = rp0 < 0 || nr < 0 || rp0 + nr > a.row_len || cp0 < 0 || nc < 0 || cp0 + nc > a.col_len;
      const int64_t n = bad ? 0 : nr + nc;
      for (int64_t i0 = tid; i0 < n; i0 += U * kBeginThreads) {
        int id[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int64_t i = min(i0 + u * kBeginThreads, n - 1);
          id[u] = i < nr ? a.row_idx[rp0 + i] : a.col_idx[cp0 + (i - nr)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) bad |= !blk::is_brief(a, id[u]);
      }
      bad = __syncthreads_or(bad);
      if (tid == 0) a.brief[b] = !bad;
    }
  }
}

}  // namespace

// Duffy rules of orders 2 .. 6 (every order the configurations use) and the
// seven-point rule have kernels of their own; the rest -- order 1 and orders
// from 7 on, whose register need grows with the order -- run the general sums,
// in the longest chunk of x-points that divides the rule (9: orders 9 and 12, 8:
// order 8, 7: order 7), else of 4 (order 8, Laplace: step of 1152 triangles 6.8 ms
// in chunks of 4, 6.0 in chunks of 8).
int rule_variant(int regular_rule, int q, int nq) {
  if (regular_rule == BEM_RULE_DUFFY && q >= 2 && q <= 6) return q;
  if (nq == 7) return blk::kSeven;
  return nq % 7 == 0 ? blk::kRule7 : nq % 9 == 0 ? blk::kRule9 : nq % 8 == 0 ? blk::kRule8 : blk::kRule4;
}

bool rule_is_duffy(int variant) { return variant < blk::kSeven; }

// Room of a column's points in LDS, in units of ypoint_doubles: one per point;
// the general sums keep ten doubles and a number per point there.
int rule_pad(int variant, int nq) {
  if (variant < blk::kRule4) return nq;
  const int xc = variant - 10;
  return std::max((nq + xc - 1) / xc * xc, 6);
}

// Default of bem_tune.x_chunk: a divisor of the rule's points.
int rule_chunk(int nq, int kernel) {
  static const int lap[] = {8, 9, 7, 5, 4};
  static const int hel[] = {4, 5, 7, 9, 8};
  for (int xc : (kernel == BEM_LAPLACE ? lap : hel))
    if (nq % xc == 0) return xc;
  return 4;
}

// LDS of a sub-tile; without the pair lists (coupling launches: every pair is
// regular, phase C only flags, and the lists sit past the allocation unread).
// slots: of the list, 0: one per pair.
size_t block_lds_bytes(int nq_pad, int tr, int tc, bool mixed, bool lists, bool both, int slots) {
  size_t dbl = (size_t)blk::ypoint_doubles(mixed) * nq_pad * tc + blk::ROW_NF * (size_t)tr +
               3 * (size_t)nq_pad + 7 * (size_t)tc + (both ? 3 * (size_t)tr : 0);
  if (mixed) dbl += 3 * (size_t)tc + 6 * (size_t)tr + 6 * (size_t)tc;
  const size_t ints = (size_t)4 * tr + 4 * (size_t)tc + 36;
  return dbl * 8 + ints * 4 + (lists ? 2 * (2 * (size_t)(slots ? slots : tr * tc) + blk::kSortPad) : 0);
}

// The limit of a requested sub-tile shape (bem_tune): not what the kernels take,
// which may shrink, but fixed, so that a stored configuration is taken or
// refused alike by every version: 48 bytes (mixed: 32) per column point, the
// rule's points rounded up to whole x_chunks, 80 bytes per row, 24 per column,
// the normals, boxes, ids and pair lists.  64 rows fit beside the default
// columns at every order, so a request of rows alone needs no check.
size_t requested_lds_bytes(int nq, int x_chunk, int tr, int tc, bool mixed, bool both) {
  const size_t r = tr, c = tc, np = (size_t)(nq + x_chunk - 1) / x_chunk * x_chunk;
  const size_t dbl = (mixed ? 4 : 6) * np * c + 10 * r + 3 * np + 3 * c + (both ? 3 * r : 0) +
                     (mixed ? 6 * r + 9 * c : 0);
  return dbl * 8 + (4 * r + 4 * c + 36) * 4 + 2 * (2 * r * c + 512);
}

// Largest sub-tile within the LDS budget.  Near-field sub-tiles carry the
// pair lists, whose entries pack row and column in 6 bits each (at most
// 64 x 64); so do mixed-precision coupling sub-tiles (their near-singular
// pairs go to the FP64 pass through the lists).  Plain coupling sub-tiles
// have no lists and take up to 128 rows and 96 columns, so that most coupling
// blocks (ranks up to ~100) are one sub-tile.
bool block_tile_shape(int nq_pad, bool mixed, size_t lds_budget, int *tr, int *tc,
                      size_t *lds_bytes, bool coupling, bool both) {
  static const int near_shapes[][2] = {{64, 64}, {64, 32}, {64, 16}, {64, 8}, {32, 8}, {16, 8},
                                       {8, 8}};
  static const int coupling_shapes[][2] = {{128, 96}, {128, 80}, {96, 80}, {128, 64}, {64, 64},
                                           {64, 32}, {64, 16}, {64, 8}, {32, 8}, {16, 8}, {8, 8}};
  const bool lists = !coupling || mixed;
  auto try_list = [&](const int(*shapes)[2], int n) {
    for (int k = 0; k < n; ++k) {
      const size_t bytes = block_lds_bytes(nq_pad, shapes[k][0], shapes[k][1], mixed, lists, both);
      if (bytes <= lds_budget) {
        *tr = shapes[k][0];
        *tc = shapes[k][1];
        *lds_bytes = bytes;
        return true;
      }
    }
    return false;
  };
  return lists ? try_list(near_shapes, 7) : try_list(coupling_shapes, 11);
}

// Workgroups per block, and narrower sub-tiles, for a launch of few blocks.
// The chip holds 512 workgroups at once (256 CUs, two by registers).  Well
// above that one workgroup per block is best: it stages a block's geometry
// once.  Below, and for the first unequal round beyond, a block's sub-tiles
// are dealt to several workgroups, so that idle CUs take part of the large
// blocks; the number is that of the mean block's sub-tiles, or twice it for
// the larger ones (any number is correct).  At most 4096 workgroups in all:
// what one reads of its whole block (the Helmholtz phase kind) stays small.
//
// Coupling blocks are mostly one sub-tile: below 768 blocks its columns are
// halved until there are 1536 (Helmholtz, order 3, 523 blocks: 436 us whole,
// 332 aiming at 1024, 267 at 1536; 632 blocks 456, 373, 331; Laplace double
// layer, 410 blocks 255, 177, 172); from 768 to 1023 blocks only the larger
// ones are dealt out (909 blocks 520 -> 472, halved too 532; 838 blocks 340 ->
// 332); 1143 blocks lose by it (572 -> 597).
// Near-field sub-tiles collect their singular pairs class by class, each class
// padded to a wave: narrower ones pay that again (mixed Helmholtz, 376 blocks:
// 420 us whole, 287 dealt out, 323 and 409 aiming at 512 and 1024 narrower
// ones).  So only lists of fewer than 320 blocks are narrowed, to 512 (64
// Laplace blocks of 64 x 64, seven points: 70 us whole, 43 aiming at 128, 29 at
// 256, 26 at 512); up to 767 blocks are dealt out (both layers, 556 blocks: 386
// -> 312; 674 blocks 377 -> 324); 1041 lose by it (1236 -> 1315).
//
// A mirrored list counts edge-adjacent pairs twice and is refused where a full
// sub-tile's pairs pass its entries.  Narrowed ones keep that limit and have the
// slots for it: their own pairs may pass their entries where the full one's do not.
void split_blocks(BlockArgs *a, bool coupling, bool mixed, bool lists, bool both, size_t *lds_bytes) {
  constexpr int64_t kDealt = 768, kDealtCoupling = 1024, kNarrow = 320, kMost = 4096;
  a->wide = a->tc;
  a->slots = a->tr * a->tc;
  a->split = 1;
  if (a->nblocks <= 0 || a->nblocks >= (coupling ? kDealtCoupling : kDealt)) return;
  const int64_t mr = std::max<int64_t>(a->row_len / a->nblocks, 1);
  const int64_t mc = std::max<int64_t>(a->col_len / a->nblocks, 1);
  const int64_t down = (mr + a->tr - 1) / a->tr;
  const bool narrow = a->nblocks < (coupling ? kDealt : kNarrow);
  const int64_t tiles = !narrow ? 0 : coupling ? 1536 : 512;
  int c = a->tc;
  while (c > 8 && a->nblocks * down * ((mc + c - 1) / c) < tiles) c = std::max(8, c / 2);
  a->tc = c;
  a->slots = std::min(2 * a->tr * c, a->tr * a->wide);
  *lds_bytes = block_lds_bytes(a->nq_pad, a->tr, c, mixed, lists, both, a->slots);
  const int64_t turns = coupling && narrow ? 1 : 2;
  a->split = (int)std::min<int64_t>(turns * down * ((mc + c - 1) / c), kMost / a->nblocks);
}

hipError_t launch_blocks(int kernel, int layer, int rule, bool coupling, bool mixed,
                         const BlockArgs &a, size_t lds, hipStream_t s) {
  if (a.nblocks == 0) return hipSuccess;
  if (kernel == BEM_LAPLACE)
    return mixed ? BlockLaunch<BEM_LAPLACE, true>::blocks(layer, rule, coupling, a, lds, s)
                 : BlockLaunch<BEM_LAPLACE, false>::blocks(layer, rule, coupling, a, lds, s);
  return mixed ? BlockLaunch<BEM_HELMHOLTZ, true>::blocks(layer, rule, coupling, a, lds, s)
               : BlockLaunch<BEM_HELMHOLTZ, false>::blocks(layer, rule, coupling, a, lds, s);
}

hipError_t launch_blocks_learned(int kernel, int layer, const BlockArgs &a, const OrderRules &o,
                                 size_t lds, hipStream_t s) {
  if (a.nblocks == 0) return hipSuccess;
  return kernel == BEM_LAPLACE ? LearnedLaunch<BEM_LAPLACE>::run(layer, a, o, lds, s)
                               : LearnedLaunch<BEM_HELMHOLTZ>::run(layer, a, o, lds, s);
}

hipError_t launch_begin(int32_t *counter, const BlockArgs *batches, int32_t nbatch, int32_t max_blocks,
                        hipStream_t s) {
  if (max_blocks == 0) {
    hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(1), 0, s, counter);
  } else {
    const dim3 grid(std::min(max_blocks, 4096), std::min(nbatch, 4096));
    hipLaunchKernelGGL(k_begin, grid, dim3(kBeginThreads), 0, s, counter, batches, nbatch);
  }
  return hipGetLastError();
}

hipError_t launch_persistent(int kernel, bool mixed, int rule, const PersistentArgs &p, size_t lds,
                             hipStream_t s) {
  if (p.ntiles == 0 || p.grid == 0) return hipSuccess;
  if (kernel == BEM_LAPLACE)
    return mixed ? PersistentLaunch<BEM_LAPLACE, true>::run(rule, p, lds, s)
                 : PersistentLaunch<BEM_LAPLACE, false>::run(rule, p, lds, s);
  return mixed ? PersistentLaunch<BEM_HELMHOLTZ, true>::run(rule, p, lds, s)
               : PersistentLaunch<BEM_HELMHOLTZ, false>::run(rule, p, lds, s);
}

}  // namespace bem
