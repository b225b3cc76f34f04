// The 32 x 256 output tile on weight words: the variants without a step list (see ring_tile.h).
#include "ring_tile.h"

template comet_gemm::GemmKernel comet_gemm::gemm_kernel_for<1, 4, 1, 2, false>(const GemmParams&);
