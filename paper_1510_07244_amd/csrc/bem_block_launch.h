// Launchers of the block kernels, one instantiation per file (bem_blocks_*.hip)
// so that they compile side by side.
#pragma once

#include <hip/hip_runtime.h>

#include "bem_internal.h"

namespace bem {

// a.nb x a.split workgroups; layer: BEM_SLP, BEM_DLP or 2 (both)
template <int KERNEL, bool MIXED>
struct BlockLaunch {
  static hipError_t blocks(int layer, int rule, bool coupling, const BlockArgs &a, size_t lds,
                           hipStream_t s);
};

template <int KERNEL, bool MIXED>
struct PersistentLaunch {
  static hipError_t run(int rule, const PersistentArgs &p, size_t lds, hipStream_t s);
};

template <int KERNEL>
struct LearnedLaunch {
  static hipError_t run(int layer, const BlockArgs &a, const OrderRules &o, size_t lds, hipStream_t s);
};

}  // namespace bem
