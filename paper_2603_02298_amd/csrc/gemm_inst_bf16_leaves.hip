// Instantiates the split and stream GEMM kernels for bf16 operands in k vectors over a k mode of several short leaves.
#include "gemm_split_kernel.hpp"
#include "gemm_stream_kernel.hpp"

namespace lc {
hipError_t launch_gemm_bf16_split_leaves(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  return launch_split_shape<true, kLoadKLeaves, kLoadKLeaves>(plan, a, b, c, s);
}
hipError_t launch_gemm_bf16_stream_leaves(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  return launch_stream_shape<true, kLoadKLeaves, kLoadKLeaves>(plan, a, b, c, s);
}
}  // namespace lc
