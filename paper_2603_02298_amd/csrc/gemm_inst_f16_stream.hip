// Instantiates the stream GEMM kernels for f16 operands.
#include "gemm_stream_kernel.hpp"

namespace lc {
hipError_t launch_gemm_f16_stream(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  return launch_stream_shape<false>(plan, a, b, c, s);
}
}  // namespace lc
