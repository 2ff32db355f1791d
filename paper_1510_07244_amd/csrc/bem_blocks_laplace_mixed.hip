// Block kernels: Laplace, the mixed form.
#include "bem_block_kernels.h"

template struct bem::BlockLaunch<BEM_LAPLACE, true>;
