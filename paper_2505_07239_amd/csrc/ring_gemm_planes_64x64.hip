// The 64 x 64 output tile of the int8 matrix-core kernel on weight planes.
#include "ring_gemm_planes.h"

template comet_gemm::GemmKernel comet_gemm::planes_kernel_for<2, 2, 2, 2, false, false>(const GemmParams&);
