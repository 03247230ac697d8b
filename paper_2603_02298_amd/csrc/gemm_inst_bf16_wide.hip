// Instantiates the wide GEMM tiles for bf16 operands.
#include "gemm_wide_kernel.hpp"

namespace lc {
hipError_t launch_gemm_bf16_wide(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  if (plan.tile_m == 256 && plan.tile_n == 192) return launch_wide<true, 4, 3>(plan, a, b, c, s);
  if (plan.tile_m == 192 && plan.tile_n == 256) return launch_wide<true, 3, 4>(plan, a, b, c, s);
  return hipErrorInvalidValue;
}
}  // namespace lc
