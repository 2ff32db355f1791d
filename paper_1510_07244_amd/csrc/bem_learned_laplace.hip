// Near field with per-entry orders: Laplace.
#include "bem_block_kernels.h"

template struct bem::LearnedLaunch<BEM_LAPLACE>;
