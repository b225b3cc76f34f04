// The grouped matrix-core kernel (several products of one shape in one launch), 128 x 64 output
// tile, weight planes: the variants for launches whose workgroups own their tiles.
#include "ring_gemm_planes.h"

template comet_gemm::GemmGroupKernel comet_gemm::planes_group_kernel_for<2, 2, 4, 2, true>(const GemmParams&);
