// Instantiates the stream GEMM kernels for f16 operands in vectors at any alignment.
#include "gemm_stream_kernel.hpp"

namespace lc {
hipError_t launch_gemm_f16_stream_any(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  return launch_stream_shape<false, kLoadKAny, kLoadRAny>(plan, a, b, c, s);
}
}  // namespace lc
