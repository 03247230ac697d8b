// Device code of the split GEMM: C(m,n) += A(m,k) * B(n,k) (Sec. 2.6.2 of "CuTe Layout Representation and Algebra") for
// problems with few tiles of C -- a thin M or N, or all three sides small -- where whole workgroups per tile leave most of the
// 256 CUs without work and the k loop is a chain of memory latencies.
//
// A workgroup of WAVES wavefronts owns a TM x TN tile of C (32 or 64 a side); its wavefronts share out the k tiles of 64
// (wavefront w takes w, w + WAVES, ...), each through a ring of STAGES tile pairs of its own that the memory pipeline fills
// straight into LDS (vectors at any alignment: one pair, filled from registers that hold the next k tile meanwhile).  Nothing is shared in the k loop, so it has no barrier: a wavefront waits for its own loads only.  The
// partial tiles are then summed through LDS in the order of the wavefronts (the same result every time) and added to C, whose
// old values were asked for before the first operand load.
// TN = 16 (at most 16 columns, contiguous along k): the 16 rows of B stand twice in their fragment, so no load is spent on
// rows that do not exist and the LDS they would take deepens the ring.
// What bounds it: the weights' way from HBM for a thin M (each element is used once), launch and latency for small problems.
// Measured on MI355X (bf16, whole 128 x 128 tiles -> this kernel): 512^3 11.1 -> 4.5 us, 16 x 8192 x 8192 78.2 -> 26.0 us
// (1.7 -> 5.2 TB/s), 1024^3 17.6 -> 8.3 us, 128 x 2048 x 2048 25.2 -> 6.4 us.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

#include "gemm_device.hpp"
#include "gemm_plan.hpp"
#include "kernarg.hpp"

namespace lc {

template <bool BF16, int TM, int TN, int WAVES, int STAGES, int A_LOAD, int B_LOAD, bool C_VEC>
__global__ __launch_bounds__(64 * WAVES) void gemm_split_kernel(GemmParams P, const uint16_t* __restrict__ A, const uint16_t* __restrict__ B,
                                                                float* __restrict__ C) {
  constexpr int FM = TM / 32, FN = (TN + 31) / 32, KSTEPS = kGemmBK / 16;
  constexpr uint32_t A_BYTES = TM * 128u, STAGE = (TM + TN) * 128u, RING = STAGES * STAGE, PARTIAL = TM * TN * 4u;
  constexpr int R = (TM + TN) / 8;   // load instructions per k tile
  constexpr bool ANY = gemm_load_in_registers(A_LOAD);
  static_assert(ANY == gemm_load_in_registers(B_LOAD), "both operands straight into LDS or both through registers");
  static_assert((A_LOAD == kLoadKLeaves) == (B_LOAD == kLoadKLeaves), "compiled for pairs");
  static_assert(TN != 16 || !gemm_load_is_k_major(B_LOAD), "16 rows: row-major tiles only");
  static_assert(PARTIAL <= RING, "a wavefront's partial tile takes the place of its own ring");
  static_assert((STAGES - 1) * R < 64, "vmcnt has six bits");
  static_assert(!ANY || STAGES == 1, "through registers: one pair of tiles");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  touch_kernel_arguments<(int)sizeof(GemmParams) + 24>();

  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const uint32_t per_batch = P.tiles_m * P.tiles_n;
  const uint32_t order = gemm_tile_order_of_block(blockIdx.x, per_batch * P.L);
  const uint32_t batch = order / per_batch;
  uint32_t tm, tn;
  gemm_tile_of_order(P, order - batch * per_batch, &tm, &tn);
  const uint32_t m0 = tm * TM, n0 = tn * TN;
  A += gemm_mode_eval(P.a_l, batch);
  B += gemm_mode_eval(P.b_l, batch);
  C += gemm_mode_eval(P.c_l, batch);

  // the C values this lane will add to: asked for first, so that they are back long before they are wanted and the waits
  // below, which count from the youngest load, never have to count them
  SumUnits<TM, TN, 64 * WAVES, C_VEC> units;
  units.request(P, C, m0, n0, tid);

  TileLoader<TM, A_LOAD, 1> la;
  TileLoader<TN, B_LOAD, 1> lb;
  init_loader<A_LOAD>(la, A, P.a_r, P.a_k, m0, P.M, P.K, lane, P.a_direct);
  init_loader<B_LOAD>(lb, B, P.b_r, P.b_k, n0, P.N, P.K, lane, P.b_direct);

  f32x16 acc[FM][FN];
  static_for<FM>([&](auto i) {
    static_for<FN>([&](auto j) {
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    });
  });

  const uint32_t ring = wave * RING;
  const uint32_t n_mine = P.k_tiles > wave ? (P.k_tiles - wave + (WAVES - 1u)) / WAVES : 0u;
  uint32_t next = n_mine > 0u ? order % n_mine : 0u;
  u32x4 af[FM][KSTEPS], bf[FN][KSTEPS];
  auto read_fragments = [&](const unsigned char* stage) {
    static_for<KSTEPS>([&](auto kk) {
      static_for<FM>([&](auto i) { af[i][kk] = direct_fragment<TM, A_LOAD>(stage, lane, 32u * (uint32_t)i, kk); });
      static_for<FN>([&](auto j) { bf[j][kk] = direct_fragment<TN, B_LOAD>(stage + A_BYTES, lane, 32u * (uint32_t)j, kk); });
    });
  };
  auto multiply = [&]() {
    static_for<KSTEPS>([&](auto kk) {
      static_for<FM>([&](auto i) {
        static_for<FN>([&](auto j) { acc[i][j] = mfma_32x32x16<BF16>(af[i][kk], bf[j][kk], acc[i][j]); });
      });
    });
  };
  if constexpr (ANY) {
    // Through registers: a k tile is parked in the wavefront's ring, the next one asked for, then its fragments are read.
    uint32_t kt = 0, asked = 0;   // the k tile being parked, the one asked for
    auto fetch = [&]() {
      asked = wave + next * WAVES;
      next = next + 1u == n_mine ? 0u : next + 1u;
      fetch_tile<A_LOAD>(la, asked, P.a_k);
      fetch_tile<B_LOAD>(lb, asked, P.b_k);
    };
    if (n_mine > 0u) fetch();
    for (uint32_t t = 0; t < n_mine; ++t) {
      unsigned char* stage = lds + ring;
      kt = asked;
      la.park(stage, kt);
      lb.park(stage + A_BYTES, kt);
      if (t + 1u < n_mine) fetch();
      __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): parked (a wavefront's LDS accesses are carried out in order)
      asm volatile("" ::: "memory");
      read_fragments(stage);
      asm volatile("" ::: "memory");
      multiply();
    }
  } else {
    auto request = [&](uint32_t at) {   // this wavefront's next k tile, to the stage at LDS offset `at`
      const uint32_t kt = wave + next * WAVES;
      next = next + 1u == n_mine ? 0u : next + 1u;
      const bool tail = kt + 1u == P.k_tiles;
      if constexpr (A_LOAD == kLoadKLeaves) {
        la.fetch(kt, P.a_k, at);
        lb.fetch(kt, P.b_k, at + A_BYTES);
      } else {
        la.fetch(2u * gemm_mode_eval(P.a_k, kt * kGemmBK), at, tail);
        lb.fetch(2u * gemm_mode_eval(P.b_k, kt * kGemmBK), at + A_BYTES, tail);
      }
    };
    static_for<STAGES>([&](auto s) {
      if ((uint32_t)s < n_mine) request(ring + (uint32_t)s * STAGE);
    });
    uint32_t at = ring;
    for (uint32_t t = 0; t < n_mine; ++t) {
      // all but the STAGES - 1 youngest k tiles have landed (vmcnt counts the newer ones; towards the end there are fewer)
      constexpr int N = (STAGES - 1) * R;
      if (t + STAGES <= n_mine) __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
      else __builtin_amdgcn_s_waitcnt(0x0F70);
      asm volatile("" ::: "memory");
      read_fragments(lds + at);
      __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): the fragments are in registers, the stage may be filled again
      asm volatile("" ::: "memory");
      if (t + STAGES < n_mine) request(at);
      multiply();
      at += STAGE;
      if (at == ring + RING) at = ring;
    }
  }

  // the partial tile, into the place of the wavefront's own ring (every load has landed and every read has returned)
  asm volatile("" ::: "memory");
  static_for<FM>([&](auto i) {
    static_for<FN>([&](auto j) {
      static_for<4>([&](auto g) {
        const uint32_t m4 = 8u * (uint32_t)i + mfma_c_row(lane, 4u * (uint32_t)g) / 4u, n = 32u * (uint32_t)j + mfma_c_col(lane);
        f32x4 v;
        static_for<4>([&](auto e) { v[(int)e] = acc[i][j][4 * g + e]; });
        if (TN >= 32 || n < (uint32_t)TN) *reinterpret_cast<f32x4*>(lds + ring + gemm_sum_unit(TM, TN, m4, n) * 16u) = v;
      });
    });
  });
  __syncthreads();
  units.add(P, C, m0, n0, tid, [&](uint32_t unit) {   // (a wavefront without a k tile left zeros)
    f32x4 part[WAVES];
    static_for<WAVES>([&](auto w) { part[w] = *reinterpret_cast<const f32x4*>(lds + (uint32_t)w * RING + unit * 16u); });
    f32x4 sum = part[0];
    static_for<WAVES - 1>([&](auto w) { sum += part[w + 1]; });
    return sum;
  });
}

template <bool BF16, int TM, int TN, int WAVES, int STAGES, int A_LOAD, int B_LOAD, bool C_VEC>
static inline hipError_t launch_split_abc(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  static_assert(WAVES * STAGES * (TM + TN) * 128 <= 160 * 1024, "the rings fit LDS");
  if (plan.lds_bytes != (unsigned)(WAVES * STAGES * (TM + TN) * 128) || plan.split_waves != WAVES) return hipErrorInvalidValue;
  static std::atomic<bool> raised{false};   // one flag per instantiation: the attribute belongs to the kernel function
  if (plan.lds_bytes > 64 * 1024 && !raised.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_split_kernel<BF16, TM, TN, WAVES, STAGES, A_LOAD, B_LOAD, C_VEC>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    raised.store(true, std::memory_order_release);
  }
  const unsigned grid = plan.params.tiles_m * plan.params.tiles_n * plan.params.L;
  hipLaunchKernelGGL((gemm_split_kernel<BF16, TM, TN, WAVES, STAGES, A_LOAD, B_LOAD, C_VEC>), dim3(grid), dim3(64 * WAVES), plan.lds_bytes, s, plan.params, a, b, c);
  return hipSuccess;
}
template <bool BF16, int TM, int TN, int WAVES, int STAGES, int A_LOAD, int B_LOAD>
static inline hipError_t launch_split_ab(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  return plan.params.c_vec ? launch_split_abc<BF16, TM, TN, WAVES, STAGES, A_LOAD, B_LOAD, true>(plan, a, b, c, s)
                           : launch_split_abc<BF16, TM, TN, WAVES, STAGES, A_LOAD, B_LOAD, false>(plan, a, b, c, s);
}
// K_LOAD, R_LOAD: the pair of load kinds (or the one kind) this translation unit holds
template <bool BF16, int TM, int TN, int WAVES, int STAGES, int K_LOAD, int R_LOAD>
static inline hipError_t launch_split(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  const int la = gemm_effective_load(plan.params.a_load, plan.params.a_direct), lb = gemm_effective_load(plan.params.b_load, plan.params.b_direct);
  if (la == K_LOAD && lb == K_LOAD) return launch_split_ab<BF16, TM, TN, WAVES, STAGES, K_LOAD, K_LOAD>(plan, a, b, c, s);
  if constexpr (K_LOAD == R_LOAD) return hipErrorInvalidValue;
  if (la == R_LOAD && lb == K_LOAD) return launch_split_ab<BF16, TM, TN, WAVES, STAGES, R_LOAD, K_LOAD>(plan, a, b, c, s);
  if constexpr (TN >= 32) {
    if (la == K_LOAD && lb == R_LOAD) return launch_split_ab<BF16, TM, TN, WAVES, STAGES, K_LOAD, R_LOAD>(plan, a, b, c, s);
    if (la == R_LOAD && lb == R_LOAD) return launch_split_ab<BF16, TM, TN, WAVES, STAGES, R_LOAD, R_LOAD>(plan, a, b, c, s);
  }
  return hipErrorInvalidValue;
}
template <bool BF16, int K_LOAD, int R_LOAD>
static inline hipError_t launch_split_shape(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  constexpr bool ANY = gemm_load_in_registers(K_LOAD);   // the k tile after the parked one waits in registers: one pair of tiles each
  if constexpr (!gemm_load_is_gather(K_LOAD) && K_LOAD != kLoadKLeaves)
    if (plan.tile_m == 32 && plan.tile_n == 16) return launch_split<BF16, 32, 16, 8, ANY ? 1 : 3, K_LOAD, R_LOAD>(plan, a, b, c, s);
  if (plan.tile_m == 32 && plan.tile_n == 32) return launch_split<BF16, 32, 32, 8, ANY ? 1 : 2, K_LOAD, R_LOAD>(plan, a, b, c, s);
  if (plan.tile_m == 32 && plan.tile_n == 64) return launch_split<BF16, 32, 64, 4, ANY ? 1 : 3, K_LOAD, R_LOAD>(plan, a, b, c, s);
  if (plan.tile_m == 64 && plan.tile_n == 32) return launch_split<BF16, 64, 32, 4, ANY ? 1 : 3, K_LOAD, R_LOAD>(plan, a, b, c, s);
  if (plan.tile_m == 64 && plan.tile_n == 64) return launch_split<BF16, 64, 64, 4, ANY ? 1 : 2, K_LOAD, R_LOAD>(plan, a, b, c, s);
  return hipErrorInvalidValue;
}

}  // namespace lc
