// The 64 x 64 output tile of the int8 matrix-core kernel on weight words: the variants that walk a step list
// (per-token row sets; see ring_words.h).
#include "ring_words.h"

template comet_gemm::GemmKernel comet_gemm::words_kernel_for<true>(const GemmParams&);
