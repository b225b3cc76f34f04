// The 64 x 64 output tile of the int8 matrix-core kernel on weight words (see ring_words.h).
#include "ring_words.h"

template comet_gemm::GemmKernel comet_gemm::words_kernel_for<false>(const GemmParams&);
