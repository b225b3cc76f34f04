// The 32 x 128 output tile of the int8 matrix-core kernel on weight planes.
#include "ring_gemm_planes.h"

template comet_gemm::GemmKernel comet_gemm::planes_kernel_for<1, 4, 2, 2, false, false>(const GemmParams&);
