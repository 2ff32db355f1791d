// Block kernels: Laplace, plain FP64.
#include "bem_block_kernels.h"

template struct bem::BlockLaunch<BEM_LAPLACE, false>;
