// Block kernels: Helmholtz, the mixed form.
#include "bem_block_kernels.h"

template struct bem::BlockLaunch<BEM_HELMHOLTZ, true>;
