// Persistent batched kernel: Helmholtz, plain FP64.
#include "bem_block_kernels.h"

template struct bem::PersistentLaunch<BEM_HELMHOLTZ, false>;
