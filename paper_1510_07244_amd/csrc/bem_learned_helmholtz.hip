// Near field with per-entry orders: Helmholtz.
#include "bem_block_kernels.h"

template struct bem::LearnedLaunch<BEM_HELMHOLTZ>;
