// The 64 x 64 output tile on weight words: the variants without a step list (see ring_tile.h).
#include "ring_tile.h"

template comet_gemm::GemmKernel comet_gemm::gemm_kernel_for<2, 2, 1, 1, false>(const GemmParams&);
