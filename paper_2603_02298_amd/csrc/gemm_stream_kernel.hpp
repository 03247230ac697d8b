// Device code of the stream GEMM: C(m,n) += A(m,k) * B(n,k) (Sec. 2.6.2 of "CuTe Layout Representation and Algebra") for
// operands that go straight into LDS, on problems with tiles for every CU but a k loop too short, or sides too small, for
// the 256 x 256 kernel, and for operands in vectors at any alignment, which pass through registers on their way into LDS.
//
// Four wavefronts own a BM x BN tile, wavefront (wm, wn) a quarter of it.  LDS holds two pairs of operand tiles; one
// barrier per k tile, after which the pair before it is overwritten by the next.  Two or more workgroups
// share a CU: one's start, its C update and its waits at the barrier lie under the others' products.  The old values of C
// are asked for before the k loop, the sums pass through LDS and C is updated in whole runs.
// What bounds it: for a short k loop C's way from and to HBM (128 x 100352 x 64: 5.4-6.3 TB/s), for a longer one the waits: for
// a k tile asked for one k tile before, for C's old values ahead of the first, at the barrier (16 x (1000 x 1504 x 776): wavefronts wait
// half of their time, matrix cores are busy 19 % of the clocks, LDS 12 %).
// Measured on MI355X (bf16, whole ring kernel of 128 x 128 tiles -> this kernel's 128 x 128): 16 x (1000 x 1504 x 776) 100 -> 83 us (in pieces of 32 k rows 82),
// a 3 x 3 convolution of 128 x 100352 x 576 39 -> 34 us (128 x 64 tiles: 32.6), 4096^3 158 -> 149 us.  Three stages and more
// (fewer workgroups per CU) measured slower wherever there are more tiles than CUs, and gained 0-7 % where there are not; so did
// 256 x 128 tiles of eight wavefronts (the batched problem 82, but 4 x 1024^3 16.5 -> 21.5) and old values of C asked for two
// units per k step (82, but 4 x 1024^3 16.5 -> 18.1).
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

#include "gemm_device.hpp"
#include "gemm_plan.hpp"
#include "kernarg.hpp"

namespace lc {

constexpr int kStreamStages = 2;   // pairs of operand tiles in LDS: one being multiplied, one on its way
constexpr int kStreamPieces = 4;   // the same LDS as pairs of 32 k rows: one being multiplied, three on their way

// PIECES (both operands k-major): k tiles of 32, four pairs in the LDS of two of 64.  The first products start after half as much and three pieces
// are under way, at the price of a barrier every 32 k: better over short k loops, worse over long ones (the rule has the figures).
template <bool BF16, int BM, int BN, int A_LOAD, int B_LOAD, bool C_VEC, bool PIECES = false>
__global__ __launch_bounds__(kBlock, 160 * 1024 / (kStreamStages * (BM + BN) * 128)) void gemm_stream_kernel(GemmParams P, const uint16_t* __restrict__ A,
                                                                                                   const uint16_t* __restrict__ B, float* __restrict__ C) {
  constexpr int FM = BM / 64, FN = BN / 64, KSTEPS = kGemmBK / 16;
  constexpr uint32_t A_BYTES = BM * 128u, STAGE = (BM + BN) * 128u;
  static_assert(BM * BN * 4 <= kStreamStages * (BM + BN) * 128, "the sums of the tile fit the ring");
  constexpr bool ANY = gemm_load_in_registers(A_LOAD);
  static_assert(ANY == gemm_load_in_registers(B_LOAD), "both operands straight into LDS or both through registers");
  static_assert((A_LOAD == kLoadKLeaves) == (B_LOAD == kLoadKLeaves), "compiled for pairs");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  touch_kernel_arguments<(int)sizeof(GemmParams) + 24>();

  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const uint32_t wm = wave & 1u, wn = wave >> 1;
  // one order over the tiles of all batch entries: an XCD (its own L2) takes a stretch of it, i.e. whole batch entries
  // where there are several, so that no operand is fetched by more XCDs than it must be
  const uint32_t per_batch = P.tiles_m * P.tiles_n;
  const uint32_t order = gemm_tile_order_of_block(blockIdx.x, per_batch * P.L);
  const uint32_t batch = order / per_batch;
  uint32_t tm, tn;
  gemm_tile_of_order(P, order - batch * per_batch, &tm, &tn);
  const uint32_t m0 = tm * BM, n0 = tn * BN;
  A += gemm_mode_eval(P.a_l, batch);
  B += gemm_mode_eval(P.b_l, batch);
  C += gemm_mode_eval(P.c_l, batch);

  static_assert(!PIECES || (A_LOAD == kLoadRDirect && B_LOAD == kLoadRDirect), "pieces of k rows: k-major tiles");
  std::conditional_t<PIECES, DirectTileLoader<BM, kLoadRDirect, 4, 32>, TileLoader<BM, A_LOAD, 4>> la;
  std::conditional_t<PIECES, DirectTileLoader<BN, kLoadRDirect, 4, 32>, TileLoader<BN, B_LOAD, 4>> lb;
  SumUnits<BM, BN, kBlock, C_VEC> units;
  // (element by element, or with k tiles on their way through registers, the old values would not leave the products the
  // registers they need: asked for at the end then)
  constexpr bool EARLY_C = C_VEC && !ANY;
  if constexpr (EARLY_C) units.request(P, C, m0, n0, tid);
  init_loader<A_LOAD>(la, A, P.a_r, P.a_k, m0, P.M, P.K, tid, P.a_direct);
  init_loader<B_LOAD>(lb, B, P.b_r, P.b_k, n0, P.N, P.K, tid, P.b_direct);

  f32x16 acc[FM][FN];
  static_for<FM>([&](auto i) {
    static_for<FN>([&](auto j) {
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    });
  });

  auto multiply = [&](const unsigned char* stage) {
    static_for<KSTEPS>([&](auto kk) {
      u32x4 af[FM], bf[FN];
      static_for<FM>([&](auto i) { af[i] = direct_fragment<BM, A_LOAD>(stage, lane, wm * (BM / 2) + 32u * (uint32_t)i, kk); });
      static_for<FN>([&](auto j) { bf[j] = direct_fragment<BN, B_LOAD>(stage + A_BYTES, lane, wn * (BN / 2) + 32u * (uint32_t)j, kk); });
      static_for<FM>([&](auto i) {
        static_for<FN>([&](auto j) { acc[i][j] = mfma_32x32x16<BF16>(af[i], bf[j], acc[i][j]); });
      });
    });
  };
  const uint32_t a_at = wave * (BM * 32u), b_at = A_BYTES + wave * (BN * 32u);   // this wavefront's quarter of either tile
  if constexpr (ANY) {
    // Through registers: k tile t + 1 is parked in the stage k tile t - 1 leaves, k tile t + 2 asked for, then k tile t multiplied.
    fetch_tile<A_LOAD>(la, 0u, P.a_k);
    fetch_tile<B_LOAD>(lb, 0u, P.b_k);
    la.park(lds + a_at, 0u);
    lb.park(lds + b_at, 0u);
    if (P.k_tiles > 1u) {
      fetch_tile<A_LOAD>(la, 1u, P.a_k);
      fetch_tile<B_LOAD>(lb, 1u, P.b_k);
    }
    for (uint32_t t = 0; t < P.k_tiles; ++t) {
      __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): parked, and the fragments of k tile t - 1 read
      lds_barrier();
      if (t + 1u < P.k_tiles) {
        unsigned char* next = lds + ((t + 1u) & 1u) * STAGE;
        la.park(next + a_at, t + 1u);
        lb.park(next + b_at, t + 1u);
        if (t + 2u < P.k_tiles) {
          fetch_tile<A_LOAD>(la, t + 2u, P.a_k);
          fetch_tile<B_LOAD>(lb, t + 2u, P.b_k);
        }
      }
      multiply(lds + (t & 1u) * STAGE);
    }
  } else if constexpr (PIECES) {
    constexpr uint32_t PIECE = (BM + BN) * 64u;
    constexpr int LOADS = BM * 32 / 512 / 4 + BN * 32 / 512 / 4, N = (kStreamPieces - 2) * LOADS;   // per piece; of the pieces behind the one that is waited for
    const uint32_t pieces = (P.K + 31u) / 32u;
    KStepOffset<32> ka, kb;   // of the next piece to request
    ka.seek(P.a_k, 0u);
    kb.seek(P.b_k, 0u);
    uint32_t asked = 0;
    auto request = [&]() {
      const bool tail = asked + 1u == pieces;
      const uint32_t at = (asked % kStreamPieces) * PIECE;
      la.fetch(ka.bytes, at + wave * (BM * 16u), tail);
      lb.fetch(kb.bytes, at + BM * 64u + wave * (BN * 16u), tail);
      ++asked;
      if (asked < pieces) {
        ka.next(P.a_k, asked);
        kb.next(P.b_k, asked);
      }
    };
    static_for<kStreamPieces - 1>([&](auto) {
      if (asked < pieces) request();
    });
    for (uint32_t t = 0; t < pieces; ++t) {
      // piece t has landed for every wavefront past the barrier, which also has its fragments of piece t - 1 in registers: that place may be
      // filled again
      if (t + kStreamPieces - 1u <= pieces) __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0070);
      else __builtin_amdgcn_s_waitcnt(0x0070);
      lds_barrier();
      if (asked < pieces) request();
      const unsigned char* piece = lds + (t % kStreamPieces) * PIECE;
      static_for<2>([&](auto kk) {
        u32x4 af[FM], bf[FN];
        static_for<FM>([&](auto i) { af[i] = direct_fragment<BM, A_LOAD>(piece, lane, wm * (BM / 2) + 32u * (uint32_t)i, kk); });
        static_for<FN>([&](auto j) { bf[j] = direct_fragment<BN, B_LOAD>(piece + BM * 64u, lane, wn * (BN / 2) + 32u * (uint32_t)j, kk); });
        static_for<FM>([&](auto i) {
          static_for<FN>([&](auto j) { acc[i][j] = mfma_32x32x16<BF16>(af[i], bf[j], acc[i][j]); });
        });
      });
    }
  } else {
    KTileOffset ka, kb;   // of the next k tile to request
    ka.seek(P.a_k, 0u);
    kb.seek(P.b_k, 0u);
    uint32_t asked = 0;
    auto request = [&](uint32_t at) {   // the next k tile, to the stage at LDS offset `at`
      const bool tail = asked + 1u == P.k_tiles;
      if constexpr (A_LOAD == kLoadKLeaves) {
        la.fetch(asked, P.a_k, at + a_at);
        lb.fetch(asked, P.b_k, at + b_at);
        ++asked;
      } else {
        la.fetch(ka.bytes, at + a_at, tail);
        lb.fetch(kb.bytes, at + b_at, tail);
        ++asked;
        if (asked < P.k_tiles) {
          ka.next(P.a_k, asked);
          kb.next(P.b_k, asked);
        }
      }
    };
    request(0u);
    for (uint32_t t = 0; t < P.k_tiles; ++t) {
      // k tile t has landed, for every wavefront past the barrier, which also has its fragments of k tile t - 1 in registers:
      // that stage may be filled again
      __builtin_amdgcn_s_waitcnt(0x0070);
      lds_barrier();
      if (asked < P.k_tiles) request((asked & 1u) * STAGE);
      multiply(lds + (t & 1u) * STAGE);
    }
  }

  __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
  lds_barrier();   // every fragment has been read: the sums take the ring's place
  static_for<FM>([&](auto i) {
    static_for<FN>([&](auto j) {
      static_for<4>([&](auto g) {
        const uint32_t m4 = wm * (BM / 8) + 8u * (uint32_t)i + mfma_c_row(lane, 4u * (uint32_t)g) / 4u;
        const uint32_t n = wn * (BN / 2) + 32u * (uint32_t)j + mfma_c_col(lane);
        f32x4 v;
        static_for<4>([&](auto e) { v[(int)e] = acc[i][j][4 * g + e]; });
        *reinterpret_cast<f32x4*>(lds + gemm_sum_unit(BM, BN, m4, n) * 16u) = v;
      });
    });
  });
  asm volatile("" ::: "memory");
  if constexpr (!EARLY_C) units.request(P, C, m0, n0, tid);   // (the products' registers are free now)
  __syncthreads();
  units.add(P, C, m0, n0, tid, [&](uint32_t unit) { return *reinterpret_cast<const f32x4*>(lds + unit * 16u); });
}

template <bool BF16, int BM, int BN, int A_LOAD, int B_LOAD, bool C_VEC, bool PIECES = false>
static inline hipError_t launch_stream_abc(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  if (plan.lds_bytes != (unsigned)(kStreamStages * (BM + BN) * 128)) return hipErrorInvalidValue;
  static std::atomic<bool> raised{false};   // one flag per instantiation: the attribute belongs to the kernel function
  if (plan.lds_bytes > 64 * 1024 && !raised.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_stream_kernel<BF16, BM, BN, A_LOAD, B_LOAD, C_VEC, PIECES>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    raised.store(true, std::memory_order_release);
  }
  const unsigned grid = plan.params.tiles_m * plan.params.tiles_n * plan.params.L;
  hipLaunchKernelGGL((gemm_stream_kernel<BF16, BM, BN, A_LOAD, B_LOAD, C_VEC, PIECES>), dim3(grid), dim3(kBlock), plan.lds_bytes, s, plan.params, a, b, c);
  return hipSuccess;
}
template <bool BF16, int BM, int BN, int A_LOAD, int B_LOAD>
static inline hipError_t launch_stream_ab(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  if constexpr (BM == 128 && BN == 128 && A_LOAD == kLoadRDirect && B_LOAD == kLoadRDirect)
    if (plan.stages == kStreamPieces)
      return plan.params.c_vec ? launch_stream_abc<BF16, BM, BN, A_LOAD, B_LOAD, true, true>(plan, a, b, c, s)
                               : launch_stream_abc<BF16, BM, BN, A_LOAD, B_LOAD, false, true>(plan, a, b, c, s);
  if (plan.stages != kStreamStages) return hipErrorInvalidValue;
  return plan.params.c_vec ? launch_stream_abc<BF16, BM, BN, A_LOAD, B_LOAD, true>(plan, a, b, c, s)
                           : launch_stream_abc<BF16, BM, BN, A_LOAD, B_LOAD, false>(plan, a, b, c, s);
}
// K_LOAD, R_LOAD: the pair of load kinds (or the one kind) this translation unit holds
template <bool BF16, int BM, int BN, int K_LOAD, int R_LOAD>
static inline hipError_t launch_stream(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  const int la = gemm_effective_load(plan.params.a_load, plan.params.a_direct), lb = gemm_effective_load(plan.params.b_load, plan.params.b_direct);
  if (la == K_LOAD && lb == K_LOAD) return launch_stream_ab<BF16, BM, BN, K_LOAD, K_LOAD>(plan, a, b, c, s);
  if constexpr (K_LOAD == R_LOAD) return hipErrorInvalidValue;
  if (la == K_LOAD && lb == R_LOAD) return launch_stream_ab<BF16, BM, BN, K_LOAD, R_LOAD>(plan, a, b, c, s);
  if (la == R_LOAD && lb == K_LOAD) return launch_stream_ab<BF16, BM, BN, R_LOAD, K_LOAD>(plan, a, b, c, s);
  if (la == R_LOAD && lb == R_LOAD) return launch_stream_ab<BF16, BM, BN, R_LOAD, R_LOAD>(plan, a, b, c, s);
  return hipErrorInvalidValue;
}
template <bool BF16, int K_LOAD, int R_LOAD>
static inline hipError_t launch_stream_shape(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  if (plan.tile_m == 128 && plan.tile_n == 128) return launch_stream<BF16, 128, 128, K_LOAD, R_LOAD>(plan, a, b, c, s);
  if (plan.tile_m == 128 && plan.tile_n == 64) return launch_stream<BF16, 128, 64, K_LOAD, R_LOAD>(plan, a, b, c, s);
  if (plan.tile_m == 64 && plan.tile_n == 128) return launch_stream<BF16, 64, 128, K_LOAD, R_LOAD>(plan, a, b, c, s);
  if (plan.tile_m == 64 && plan.tile_n == 64) return launch_stream<BF16, 64, 64, K_LOAD, R_LOAD>(plan, a, b, c, s);
  return hipErrorInvalidValue;
}

}  // namespace lc
