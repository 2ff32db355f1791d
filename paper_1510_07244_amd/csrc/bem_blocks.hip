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

}  // namespace

// Duffy rules of orders 2 .. 6 have kernels of their own (every order the
// configurations use); the rest -- seven points per triangle, order 1 and
// orders from 7 on, whose register need grows with the order -- run the
// general sums in chunks of 7 x-points, or of 4 with padding.
int rule_variant(int regular_rule, int q, int nq) {
  if (regular_rule == BEM_RULE_DUFFY && q >= 2 && q <= 6) return q;
  return nq % 7 == 0 ? blk::kRule7 : blk::kRule4;
}

int rule_pad(int variant, int nq) {
  if (variant < blk::kRule4) return nq;
  const int xc = variant - 10;
  return (nq + xc - 1) / xc * xc;
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
size_t block_lds_bytes(int nq_pad, int tr, int tc, bool mixed, bool lists, bool both) {
  size_t dbl = (size_t)blk::ypoint_doubles(mixed) * nq_pad * tc + blk::ROW_NF * (size_t)tr +
               3 * (size_t)nq_pad + 7 * (size_t)tc + (both ? 3 * (size_t)tr : 0);
  if (mixed) dbl += 3 * (size_t)tc + 6 * (size_t)tr + 6 * (size_t)tc;
  const size_t ints = (size_t)4 * tr + 4 * (size_t)tc + 36;
  return dbl * 8 + ints * 4 + (lists ? (size_t)2 * (2 * (size_t)tr * tc + blk::kSortPad) : 0);
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
// The chip holds 512 workgroups at once (256 CUs, two by registers); from
// that many blocks on, one workgroup each is better (it stages a block's
// geometry once).  Below it a block's sub-tiles are dealt to several
// workgroups, and their columns halved (to 8 at the least, which still gives
// every thread an entry per pass) until the list has about 1024 sub-tiles:
// two rounds, so that unequal ones even out.  The number of sub-tiles is the
// mean block's; any split is correct, larger blocks give their workgroups
// several turns.  At most 4096 workgroups in all: what a workgroup reads of
// its whole block (the Helmholtz phase kind) stays small.
// 64 Laplace blocks of 64 x 64, seven points, both kinds of split: 70 -> 25 us;
// double layer, order 5: 420 -> 111; mixed Helmholtz coupling, 64 blocks:
// 497 -> 158; near field in 376 blocks: 231 -> 191; aiming at 512 or 2048
// sub-tiles instead: 183 / 160 against 156 us for 419 coupling blocks; the
// split from 880 blocks on instead of below 512: 1318 -> 1870 us.
int split_blocks(const BlockArgs &a, bool mixed, bool lists, bool both, int *tc, size_t *lds_bytes) {
  constexpr int64_t kFull = 512, kTiles = 1024, kMost = 4096;
  if (a.nblocks >= kFull || a.nblocks <= 0) return 1;
  const int64_t mr = std::max<int64_t>(a.row_len / a.nblocks, 1);
  const int64_t mc = std::max<int64_t>(a.col_len / a.nblocks, 1);
  const int64_t down = (mr + a.tr - 1) / a.tr;
  int c = *tc;
  while (c > 8 && a.nblocks * down * ((mc + c - 1) / c) < kTiles) c = std::max(8, c / 2);
  *tc = c;
  *lds_bytes = block_lds_bytes(a.nq_pad, a.tr, c, mixed, lists, both);
  return (int)std::min<int64_t>(down * ((mc + c - 1) / c), kMost / a.nblocks);
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

hipError_t launch_reset_counter(int32_t *counter, hipStream_t s) {
  hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(1), 0, s, counter);
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
