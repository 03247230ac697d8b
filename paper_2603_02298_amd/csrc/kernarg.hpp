// Kernel arguments live in memory; this is how the kernels bring all of their lines in at once.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace lc {

// Reads one dword of every 64-byte line of the kernel-argument block, all at once.  The blocks here
// span up to a dozen lines and their fields are needed one group after the other; without this
// each group's first use pays its own scalar-cache miss, in series, before the first global load.
template <int BYTES>
__device__ __forceinline__ void touch_kernel_arguments() {
  typedef const uint32_t __attribute__((address_space(4))) * KernargPtr;
  KernargPtr ka = (KernargPtr)__builtin_amdgcn_kernarg_segment_ptr();
  constexpr int LINES = (BYTES + 63) / 64;
  static_assert(LINES <= 16, "one scalar register per line");
  uint32_t t[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) t[i] = ka[(i < LINES ? i : 0) * 16];
  // a use the compiler cannot move or split: all loads are issued together, and waited for, here
  asm volatile("" ::"s"(t[0]), "s"(t[1]), "s"(t[2]), "s"(t[3]), "s"(t[4]), "s"(t[5]), "s"(t[6]), "s"(t[7]), "s"(t[8]), "s"(t[9]),
               "s"(t[10]), "s"(t[11]), "s"(t[12]), "s"(t[13]), "s"(t[14]), "s"(t[15]));
}

}  // namespace lc
