// Instantiates the stream GEMM kernels for f16 operands that go straight into LDS.
#include "gemm_stream_kernel.hpp"

namespace lc {
hipError_t launch_gemm_f16_stream(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  return launch_stream_shape<false, kLoadKDirect, kLoadRDirect>(plan, a, b, c, s);
}
}  // namespace lc
