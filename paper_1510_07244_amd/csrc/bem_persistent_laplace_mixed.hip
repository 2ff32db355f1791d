// Persistent batched kernel: Laplace, the mixed form.
#include "bem_block_kernels.h"

template struct bem::PersistentLaunch<BEM_LAPLACE, true>;
