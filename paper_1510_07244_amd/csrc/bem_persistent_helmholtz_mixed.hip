// Persistent batched kernel: Helmholtz, the mixed form.
#include "bem_block_kernels.h"

template struct bem::PersistentLaunch<BEM_HELMHOLTZ, true>;
