// Instantiates the split GEMM kernels for bf16 operands that go straight into LDS.
#include "gemm_split_kernel.hpp"

namespace lc {
hipError_t launch_gemm_bf16_split(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  return launch_split_shape<true, kLoadKDirect, kLoadRDirect>(plan, a, b, c, s);
}
}  // namespace lc
