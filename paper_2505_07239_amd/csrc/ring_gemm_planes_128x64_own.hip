// The 128 x 64 output tile of the int8 matrix-core kernel on weight planes: the variants for
// launches whose workgroups own their tiles.
#include "ring_gemm_planes.h"

template comet_gemm::GemmKernel comet_gemm::planes_kernel_for<2, 2, 4, 2, false, true>(const GemmParams&);
