// Device code of the wide GEMM tiles: C(m,n) += A(m,k) * B(n,k) (Sec. 2.6.2 of "CuTe Layout Representation and Algebra") for
// operands that go straight into LDS and a C with vectors, in tiles of 256 x 192 or 192 x 256, one workgroup a CU.
//
// The main loop is the ring of five operand tiles of gemm_kernel.hpp, described there (slots as large as the larger tile): its counted waits, the order of
// its loads and its slots are the same in both, and a change to one is due in the other.  (Both through one function: the same sums, but
// the registers fall differently, 256 x 256 tiles 1.010 of the time over 52 problems, 256 x 192 1.009 over 44.)
// The 256 x 256 tiles read least of LDS and memory per product, but on problems with one to four of them a CU the last round is often
// mostly empty; these are the next best per product (192 sums a lane still leave the fragments double-buffered) and fill the rounds differently.
// What bounds it: the matrix cores at the power limit inside the loop, C's way from and to HBM behind it, which nothing covers.
// Measured on MI355X (bf16, us; best of the other tiles -> this): nt 3368 x 5336 x 6576 334 -> 299, tt 3144 x 6368 x 3992 241 -> 212,
// tt 5656 x 2968 x 8048 380 -> 311, nt 4272 x 3896 x 3376 183 -> 164, tt 1200 x 7016 x 1432 49 -> 41; where 256 x 256 fills its rounds it
// stays ahead (4096^3 134, 184 here).  C's old values asked for under the first k tiles' products do not fit the registers beside
// the sums (10 spills for a third of them: 3144 x 6368 x 3992 212 -> 218).
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

#include "gemm_device.hpp"
#include "gemm_plan.hpp"
#include "kernarg.hpp"

namespace lc {

template <bool BF16, int WMB, int WNB, int A_LOAD, int B_LOAD>
__global__ __launch_bounds__(kBlock, 1) void gemm_wide_kernel(GemmParams P, const uint16_t* __restrict__ A, const uint16_t* __restrict__ B,
                                                              float* __restrict__ C) {
  constexpr int BM = 64 * WMB, BN = 64 * WNB, KSTEPS = kGemmBK / 16;
  constexpr uint32_t SLOT = (BM > BN ? BM : BN) * 128u;
  constexpr int RA = BM / 32, RB = BN / 32, MFMAS = WMB * WNB;   // load instructions per lane and operand tile
  constexpr int DS_READS = WMB * (A_LOAD == kLoadRDirect ? 2 : 1) + WNB * (B_LOAD == kLoadRDirect ? 2 : 1);
  static_assert(KSTEPS == 4, "the loop below spells out the four k steps");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  touch_kernel_arguments<(int)sizeof(GemmParams) + 24>();

  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const uint32_t wm = wave & 1u, wn = wave >> 1;
  const uint32_t per_batch = P.tiles_m * P.tiles_n;
  const uint32_t order = gemm_tile_order_of_block(blockIdx.x, per_batch * P.L);
  const uint32_t batch = order / per_batch;
  uint32_t tm, tn;
  gemm_tile_of_order(P, order - batch * per_batch, &tm, &tn);
  const uint32_t m0 = tm * BM, n0 = tn * BN;
  A += gemm_mode_eval(P.a_l, batch);
  B += gemm_mode_eval(P.b_l, batch);
  C += gemm_mode_eval(P.c_l, batch);

  DirectTileLoader<BM, A_LOAD, 4> la;
  DirectTileLoader<BN, B_LOAD, 4> lb;
  la.init(A, P.a_r, P.a_k, m0, P.M, P.K, tid);
  lb.init(B, P.b_r, P.b_k, n0, P.N, P.K, tid);
  const uint32_t a_own = wave * (RA * 1024u), b_own = wave * (RB * 1024u);   // this wavefront's share of a slot

  const uint32_t last = P.k_tiles - 1u;
  KTileOffset ka, kb;   // of the newest k tile requested for A and for B
  ka.seek(P.a_k, 0u);
  kb.seek(P.b_k, 0u);
  la.fetch(ka.bytes, 0u * SLOT + a_own, last == 0u);
  lb.fetch(kb.bytes, 1u * SLOT + b_own, last == 0u);
  __builtin_amdgcn_sched_barrier(0x038F);   // k tile 0's loads stay the oldest: the first wait below counts from the youngest
  ka.seek(P.a_k, last < 1u ? last : 1u);
  kb.seek(P.b_k, last < 1u ? last : 1u);
  la.fetch(ka.bytes, 2u * SLOT + a_own, last <= 1u);
  lb.fetch(kb.bytes, 3u * SLOT + b_own, last <= 1u);
  ka.seek(P.a_k, last < 2u ? last : 2u);
  la.fetch(ka.bytes, 4u * SLOT + a_own, last <= 2u);

  f32x16 acc[WMB][WNB];
  static_for<WMB>([&](auto i) {
    static_for<WNB>([&](auto j) {
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    });
  });
  // per fragment: the lane's LDS address for the tile's first k step in the slot being multiplied.  Row-major tiles: k step
  // kk flips slot bits (address ^ 32 kk); k-major tiles: k step kk is a constant offset.
  u32x4 af[2][WMB], bf[2][WNB];
  uint32_t a_fr[WMB], b_fr[WNB];
  static_for<WMB>([&](auto i) {
    const uint32_t row = wm * (WMB * 32u) + 32u * (uint32_t)i;
    a_fr[i] = A_LOAD == kLoadRDirect ? gemm_rdirect_frag_offset(BM, lane, row, 8u * mfma_ab_kvec(lane)) : gemm_lds_offset(row + mfma_ab_row(lane), mfma_ab_kvec(lane));
  });
  static_for<WNB>([&](auto j) {
    const uint32_t row = wn * (WNB * 32u) + 32u * (uint32_t)j;
    b_fr[j] = SLOT + (B_LOAD == kLoadRDirect ? gemm_rdirect_frag_offset(BN, lane, row, 8u * mfma_ab_kvec(lane)) : gemm_lds_offset(row + mfma_ab_row(lane), mfma_ab_kvec(lane)));
  });
  auto read_fragments = [&](auto kk, auto buf) {
    static_for<WMB>([&](auto i) {
      if constexpr (A_LOAD == kLoadRDirect) af[buf][i] = lds_read_tr_16x8<BM>(lds + a_fr[i], kk);
      else af[buf][i] = *reinterpret_cast<const u32x4*>(lds + (a_fr[i] ^ (32u * (uint32_t)kk)));
    });
    static_for<WNB>([&](auto j) {
      if constexpr (B_LOAD == kLoadRDirect) bf[buf][j] = lds_read_tr_16x8<BN>(lds + b_fr[j], kk);
      else bf[buf][j] = *reinterpret_cast<const u32x4*>(lds + (b_fr[j] ^ (32u * (uint32_t)kk)));
    });
  };
  auto multiply = [&](auto buf) {
    static_for<WMB>([&](auto i) {
      static_for<WNB>([&](auto j) { acc[i][j] = mfma_32x32x16<BF16>(af[buf][i], bf[buf][j], acc[i][j]); });
    });
  };
  // issue order inside a k step: its loads and LDS reads spread evenly between the MFMAs (the reads over the first `span` of them)
  auto issue_order = [&](auto loads_c, auto span_c) {
    constexpr int LOADS = loads_c, SPAN = span_c;
    static_for<MFMAS>([&](auto g) {
      constexpr int loads = LOADS * (g + 1) / MFMAS - LOADS * g / MFMAS;
      constexpr int reads = g < SPAN ? DS_READS * (g + 1) / SPAN - DS_READS * g / SPAN : 0;
      if constexpr (loads > 0) __builtin_amdgcn_sched_group_barrier(0x010, loads, 0);
      if constexpr (reads > 0) __builtin_amdgcn_sched_group_barrier(0x100, reads, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    });
  };
  auto next_slot = [](uint32_t slot) { return slot + 2u >= 5u ? slot + 2u - 5u : slot + 2u; };
  // s_waitcnt vmcnt(n) lgkmcnt(0): all but the n youngest loads have landed, every LDS read has returned
  auto wait_loads_but = [](auto n) {
    constexpr int N = decltype(n)::value;
    static_assert(N >= 0 && N < 64, "vmcnt has six bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0070);
  };
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  wait_loads_but(std::integral_constant<int, 2 * RA + RB>{});   // k tile 0 has landed
  lds_barrier();
  read_fragments(I0{}, I0{});
  uint32_t sa = 0u, sb = 1u;   // slots of the k tile being multiplied
  for (uint32_t kt = 0; kt < P.k_tiles; ++kt) {
    const uint32_t s_b1 = next_slot(sb), s_a2 = next_slot(next_slot(sa));   // slots of B(kt + 1) and A(kt + 2)
    const bool b1_last = kt + 1u >= last, a2_last = kt + 2u >= last;
    lb.template fetch<RB / 2, RB>(kb.bytes, s_b1 * SLOT + b_own, b1_last);
    read_fragments(I1{}, I1{});
    multiply(I0{});
    issue_order(std::integral_constant<int, RB - RB / 2>{}, std::integral_constant<int, MFMAS>{});
    // the wait before the barrier counts loads: nothing but A(kt + 2)'s may be scheduled behind this
    __builtin_amdgcn_sched_barrier(0x038F);
    la.template fetch<0, RA / 2>(ka.bytes, s_a2 * SLOT + a_own, a2_last);
    read_fragments(std::integral_constant<int, 2>{}, I0{});
    multiply(I1{});
    issue_order(std::integral_constant<int, RA / 2>{}, std::integral_constant<int, MFMAS>{});
    la.template fetch<RA / 2, RA>(ka.bytes, s_a2 * SLOT + a_own, a2_last);
    read_fragments(std::integral_constant<int, 3>{}, I1{});
    multiply(I0{});
    issue_order(std::integral_constant<int, RA - RA / 2>{}, std::integral_constant<int, (MFMAS + 1) / 2>{});
    wait_loads_but(std::integral_constant<int, RA>{});   // k tile kt + 1 has landed; A(kt + 2) may still be on its way
    lds_barrier();
    if (kt + 2u <= last) kb.next(P.b_k, kt + 2u);
    if (kt + 3u <= last) ka.next(P.a_k, kt + 3u);
    // k step 3: first half of B(kt + 2), into the slot A(kt) leaves
    lb.template fetch<0, RB / 2>(kb.bytes, sa * SLOT + b_own, a2_last);
    const uint32_t sa_next = next_slot(sa), sb_next = next_slot(sb);
    const uint32_t da = (sa_next - sa) * SLOT, db = (sb_next - sb) * SLOT;
    static_for<WMB>([&](auto i) { a_fr[i] += da; });
    static_for<WNB>([&](auto j) { b_fr[j] += db; });
    sa = sa_next;
    sb = sb_next;
    read_fragments(I0{}, I0{});
    multiply(I1{});
    issue_order(std::integral_constant<int, RB / 2>{}, std::integral_constant<int, MFMAS>{});
  }

  // C(m,n) += acc: every vector asked for before the first is stored; entries that do not exist read the last ones that do
  uint32_t c_row[WMB][4], c_col[WNB];
  static_for<WMB>([&](auto i) {
    static_for<4>([&](auto g) {
      const uint32_t m = m0 + wm * (WMB * 32u) + 32u * (uint32_t)i + mfma_c_row(lane, 4u * (uint32_t)g);
      c_row[i][g] = gemm_mode_eval(P.c_m, m < P.M ? m : P.M - 4u);
    });
  });
  static_for<WNB>([&](auto j) {
    const uint32_t n = n0 + wn * (WNB * 32u) + 32u * (uint32_t)j + mfma_c_col(lane);
    c_col[j] = gemm_mode_eval(P.c_n, n < P.N ? n : P.N - 1u);
  });
  f32x4 old[WNB][WMB][4];
  static_for<WNB>([&](auto j) {
    static_for<WMB>([&](auto i) {
      static_for<4>([&](auto g) { old[j][i][g] = *reinterpret_cast<const f32x4*>(C + (c_row[i][g] + c_col[j])); });
    });
  });
  static_for<WNB>([&](auto j) {
    const uint32_t n = n0 + wn * (WNB * 32u) + 32u * (uint32_t)j + mfma_c_col(lane);
    static_for<WMB>([&](auto i) {
      static_for<4>([&](auto g) {
        const uint32_t m = m0 + wm * (WMB * 32u) + 32u * (uint32_t)i + mfma_c_row(lane, 4u * (uint32_t)g);
        f32x4 c = old[j][i][g];
        static_for<4>([&](auto v) { c[(int)v] += acc[i][j][4 * g + v]; });
        if (n < P.N && m < P.M) *reinterpret_cast<f32x4*>(C + (c_row[i][g] + c_col[j])) = c;
      });
    });
  });
  __builtin_amdgcn_s_waitcnt(0x0F70);   // the repeated loads of the last k tile end before the wavefront does
}

template <bool BF16, int WMB, int WNB, int A_LOAD, int B_LOAD>
static inline hipError_t launch_wide_ab(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  if (plan.lds_bytes != 5u * 256u * 128u || !plan.params.c_vec) return hipErrorInvalidValue;
  static std::atomic<bool> raised{false};   // one flag per instantiation: the attribute belongs to the kernel function
  if (!raised.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_wide_kernel<BF16, WMB, WNB, A_LOAD, B_LOAD>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    raised.store(true, std::memory_order_release);
  }
  const unsigned grid = plan.params.tiles_m * plan.params.tiles_n * plan.params.L;
  hipLaunchKernelGGL((gemm_wide_kernel<BF16, WMB, WNB, A_LOAD, B_LOAD>), dim3(grid), dim3(kBlock), plan.lds_bytes, s, plan.params, a, b, c);
  return hipSuccess;
}
template <bool BF16, int WMB, int WNB>
static inline hipError_t launch_wide(const lc_gemm_plan& plan, const uint16_t* a, const uint16_t* b, float* c, hipStream_t s) {
  const int la = gemm_effective_load(plan.params.a_load, plan.params.a_direct), lb = gemm_effective_load(plan.params.b_load, plan.params.b_direct);
  if (la == kLoadKDirect && lb == kLoadKDirect) return launch_wide_ab<BF16, WMB, WNB, kLoadKDirect, kLoadKDirect>(plan, a, b, c, s);
  if (la == kLoadKDirect && lb == kLoadRDirect) return launch_wide_ab<BF16, WMB, WNB, kLoadKDirect, kLoadRDirect>(plan, a, b, c, s);
  if (la == kLoadRDirect && lb == kLoadKDirect) return launch_wide_ab<BF16, WMB, WNB, kLoadRDirect, kLoadKDirect>(plan, a, b, c, s);
  if (la == kLoadRDirect && lb == kLoadRDirect) return launch_wide_ab<BF16, WMB, WNB, kLoadRDirect, kLoadRDirect>(plan, a, b, c, s);
  return hipErrorInvalidValue;
}

}  // namespace lc
