// Instantiates the split and stream GEMM kernels for f16 operands without vectors, or with vectors over any k mode.
#include "gemm_split_kernel.hpp"
#include "gemm_stream_kernel.hpp"

namespace lc {
hipError_t launch_gemm_f16_split_gather(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  return launch_split_shape<false, kLoadKGather, kLoadRGather>(plan, a, b, c, s);
}
hipError_t launch_gemm_f16_stream_gather(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  return launch_stream_shape<false, kLoadKGather, kLoadRGather>(plan, a, b, c, s);
}
}  // namespace lc
