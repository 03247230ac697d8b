// Instantiates the split GEMM kernels for f16 operands in vectors at any alignment.
#include "gemm_split_kernel.hpp"

namespace lc {
hipError_t launch_gemm_f16_split_any(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  return launch_split_shape<false, kLoadKAny, kLoadRAny>(plan, a, b, c, s);
}
}  // namespace lc
