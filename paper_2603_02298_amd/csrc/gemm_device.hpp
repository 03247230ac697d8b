// Device helpers the GEMM kernels share: the matrix instruction, register transposes, LDS transpose loads, the barrier and
// the step along an operand's k mode.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "gemm_params.hpp"

namespace lc {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

template <bool BF16>
__device__ __forceinline__ f32x16 mfma_32x32x16(u32x4 a, u32x4 b, f32x16 c) {
  if constexpr (BF16)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// Row i of the transpose of an 8x8 block of 16-bit elements held as 8 vectors of 8 (in[j] = the 8 rows' elements
// at column j): element j of the result is element i of in[j].  `odd` says whether i is odd (it may be a run-time
// value: it only picks the halves of the dwords, never a register); half = i / 2 picks the dword.
__device__ __forceinline__ u32x4 transposed_row_b16(const u32x4 (&in)[8], int half, bool odd) {
  // v_perm_b32 picks 4 of the 8 bytes {in[2d+1] dword : in[2d] dword}: low halves of both, or high halves of both
  const uint32_t sel = odd ? 0x07060302u : 0x05040100u;
  u32x4 out;
#pragma unroll
  for (int d = 0; d < 4; ++d) out[d] = __builtin_amdgcn_perm(in[2 * d + 1][half], in[2 * d][half], sel);
  return out;
}

// compile-time loop: f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>); the accumulators are
// only ever indexed with constants, so they stay in registers
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// One 32 x 16 fragment's share of a lane from a k-major tile (row k of the tile = BR elements, see gemm_rdirect_lds_offset):
// two LDS transpose loads (ds_read_b64_tr_b16) of k .. k + 3 and k + 4 .. k + 7; `at` is the lane's address for the
// tile's first 16 k, kk the k step.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
// The restrict qualifier gives the load alias information once inlined; without any, the compiler makes every such load wait
// for all direct loads in flight (they write LDS too), although those go to the other stage.
__device__ __forceinline__ s16x4 lds_transpose_load(lds_s16x4* __restrict__ p) { return __builtin_amdgcn_ds_read_tr16_b64_v4i16(p); }
template <int BR, typename KK>
__device__ __forceinline__ u32x4 lds_read_tr_16x8(const unsigned char* at, KK kk) {
  const unsigned char* p = at + (uint32_t)kk * 16u * (BR * 2u);
  const s16x4 lo = lds_transpose_load((lds_s16x4*)(p));
  const s16x4 hi = lds_transpose_load((lds_s16x4*)(p + 4u * (BR * 2u)));
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 l = __builtin_bit_cast(u32x2, lo), h = __builtin_bit_cast(u32x2, hi);
  return u32x4{l[0], l[1], h[0], h[1]};
}

__device__ __forceinline__ u32x4 select_or_zero(bool keep, u32x4 v) {
  return u32x4{keep ? v[0] : 0u, keep ? v[1] : 0u, keep ? v[2] : 0u, keep ? v[3] : 0u};
}

// Workgroup barrier that orders LDS accesses only.  __syncthreads() would also wait for every load in flight (the direct
// loads count as global loads), which is exactly what the ring of tiles must not do; the caller states its own wait.
__device__ __forceinline__ void lds_barrier() {
  // the empty statements are compiler-only fences: no memory access is moved across the barrier, nothing is emitted
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Byte offset of k tile t along an operand's k mode, for operands whose k tiles lie inside the mode's first leaf: stepping
// to the next tile adds 64 strides of that leaf until the leaf is exhausted; only then is the layout function evaluated again.
template <int BK>   // k extent of a tile
struct KStepOffset {
  uint32_t bytes, step, left;   // left: k tiles from the current one to the end of the first leaf's run
  __device__ __forceinline__ void seek(const GemmMode& k, uint32_t t) {
    bytes = 2u * gemm_mode_eval(k, t * BK);
    step = 2u * BK * k.lead_stride;
    if (k.n == 1) {
      left = 0xFFFFFFFFu;
    } else {
      uint32_t q, r;
      fd_divmod(t * BK, k.div[0], &q, &r);
      left = (k.div[0].div - r) / BK;
    }
  }
  __device__ __forceinline__ void next(const GemmMode& k, uint32_t t) {
    if (--left == 0) seek(k, t);
    else bytes += step;
  }
};
using KTileOffset = KStepOffset<kGemmBK>;

// One operand's tile of a k tile sent straight from global memory into LDS by WAVES wavefronts together: R instructions of
// 1 KiB per wavefront (lane t's 16 bytes land at byte 16 t of the KiB).
// Rows past the operand's extent, and k past K in a short last k tile, present an offset outside the buffer's range: zeros
// arrive and no access is made.
// BK: k extent of the tile (32: k-major tiles only, a piece of 32 k rows)
template <int BR, int LOAD, int WAVES, int BK = kGemmBK>
struct DirectTileLoader {
  static constexpr int R = BR * BK / 512 / WAVES;
  static_assert(BK == kGemmBK || LOAD == kLoadRDirect, "row-major tiles hold whole rows of 64");
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t off[R];       // bytes from the k tile's first k
  uint32_t tail_mask;    // bit i: instruction i of this lane asks for k below K in the last k tile

  // t: the lane's index among the WAVES wavefronts' lanes
  __device__ __forceinline__ void init(const uint16_t* p, const GemmMode& rmode, const GemmMode& kmode, uint32_t row0, uint32_t extent, uint32_t K,
                                       uint32_t t) {
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p), 0, 0xFFFFFFFFu, 0x00020000);
    tail_mask = 0u;
    const uint32_t k_rem = K - (K - 1u) / BK * BK;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      uint32_t row, k, in_k;   // in_k: elements from the k tile's first k
      if constexpr (LOAD == kLoadKDirect) {
        row = gemm_direct_row(R, t, (uint32_t)i);
        k = 8u * gemm_direct_kvec(row, t);
        in_k = k;
      } else {
        gemm_rdirect_unit(BR, R, t, (uint32_t)i, &k, &row);
        in_k = k * kmode.lead_stride;
      }
      const uint32_t r = row0 + row, at = 2u * (gemm_mode_eval(rmode, r < extent ? r : extent - 1u) + in_k);
      off[i] = r < extent ? at : 0xFFFFFFFFu;
      tail_mask |= (k < k_rem ? 1u : 0u) << i;
    }
  }
  // k_bytes: the k tile's byte offset along the k mode (uniform); at: where this wavefront's first KiB of the tile lies in LDS (uniform);
  // FIRST, END: which of the instructions
  template <int FIRST = 0, int END = R>
  __device__ __forceinline__ void fetch(uint32_t k_bytes, uint32_t at, bool tail) {
    typedef __attribute__((address_space(3))) void lds_void;
    // dynamic LDS under a second name: the compiler sees no alias between these writes and the fragment reads and adds no
    // waits of its own; the kernels state the order by hand
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_bytes[];
    static_for<END - FIRST>([&](auto d) {
      constexpr int i = FIRST + decltype(d)::value;
      const uint32_t voff = (tail && ((tail_mask >> i) & 1u) == 0u) ? 0xFFFFFFFFu : off[i];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)(lds_bytes + at + (uint32_t)i * 1024u), 16, (int)voff, (int)k_bytes, 0, 0);
    });
  }
};

// The same over any k mode whose first leaf holds whole vectors: lane l evaluates the mode for k vector l % 8 of the tile, the
// others read it from there.  (Measured on MI355X, us; staged through registers -> this: convolutions of 128 x 90750 x 144 47 -> 22.6, of
// 232 x 33856 x 288 30.6 -> 21.9; in vectors gathered through registers 256 x 115200 x 288 takes 80, this 67-70.)
template <int BR, int WAVES>
struct LeavesTileLoader {
  static constexpr int R = BR / 8 / WAVES;
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t off[R];       // bytes of the lane's row; 0xFFFFFFFF: no such row
  uint32_t K, t;
  __device__ __forceinline__ void init(const uint16_t* p, const GemmMode& rmode, const GemmMode&, uint32_t row0, uint32_t extent, uint32_t Ktot, uint32_t lane) {
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p), 0, 0xFFFFFFFFu, 0x00020000);
    K = Ktot;
    t = lane;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const uint32_t r = row0 + gemm_direct_row(R, t, (uint32_t)i);
      off[i] = r < extent ? 2u * gemm_mode_eval(rmode, r) : 0xFFFFFFFFu;
    }
  }
  __device__ __forceinline__ void fetch(uint32_t kt, const GemmMode& kmode, uint32_t at) {
    typedef __attribute__((address_space(3))) void lds_void;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_bytes[];   // (see DirectTileLoader)
    const uint32_t k0 = kt * kGemmBK, mine = k0 + 8u * (t & 7u);
    const uint32_t k_off = mine < K ? 2u * gemm_mode_eval(kmode, mine) : 0xFFFFFFFFu;
    static_for<R>([&](auto i) {
      const uint32_t kv = gemm_direct_kvec(gemm_direct_row(R, t, (uint32_t)i), t);
      const uint32_t theirs = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(4u * kv), (int)k_off);
      const uint32_t voff = off[i] != 0xFFFFFFFFu && theirs != 0xFFFFFFFFu ? off[i] + theirs : 0xFFFFFFFFu;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)(lds_bytes + at + (uint32_t)i * 1024u), 16, (int)voff, 0, 0, 0);
    });
  }
};

// The 8 elements of v moved down by n elements (0 .. 8), zeros from above.
__device__ __forceinline__ u32x4 move_down_b16(u32x4 v, uint32_t n) {
  uint64_t lo = (uint64_t)v[0] | ((uint64_t)v[1] << 32), hi = (uint64_t)v[2] | ((uint64_t)v[3] << 32);
  if (n >= 4u) { lo = hi; hi = 0u; }
  const uint32_t bits = 16u * (n & 3u);
  lo = bits ? (lo >> bits) | (hi << (64u - bits)) : lo;
  hi >>= bits;
  if (n >= 8u) lo = hi = 0u;
  return u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
}

// The same tile brought in through registers, for operands whose vectors lie at any 2-byte-aligned address (kLoadKAny,
// kLoadRAny): the units a lane loads and where they lie in LDS are those of the direct loads.
template <int BR, int LOAD, int WAVES>
struct AnyTileLoader {
  static constexpr int R = BR / 8 / WAVES;
  typedef u32x4 __attribute__((aligned(2))) u32x4_any;
  const unsigned char* base;
  uint32_t off[R];       // bytes from the k tile's first k
  uint32_t K, k_step, row0, extent, t;   // k_step: bytes from one k to the next
  u32x4 regs[R];

  // unit i of this lane: its row, and its k inside the k tile (along k: of its first element)
  __device__ __forceinline__ void unit(uint32_t i, uint32_t* row, uint32_t* k) const {
    if constexpr (LOAD == kLoadKAny) {
      *row = gemm_direct_row(R, t, i);
      *k = 8u * gemm_direct_kvec(*row, t);
    } else {
      gemm_rdirect_unit(BR, R, t, i, k, row);
    }
  }
  __device__ __forceinline__ void init(const uint16_t* p, const GemmMode& rmode, const GemmMode& kmode, uint32_t first_row, uint32_t rows, uint32_t Ktot,
                                       uint32_t lane) {
    base = reinterpret_cast<const unsigned char*>(p);
    K = Ktot;
    k_step = 2u * kmode.lead_stride;
    row0 = first_row;
    extent = rows;
    t = lane;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      uint32_t row, k;
      unit((uint32_t)i, &row, &k);
      off[i] = gemm_any_offset(LOAD, rmode, row0 + row, extent, k, K, k_step);
    }
  }
  // asks for k tile kt
  __device__ __forceinline__ void fetch(uint32_t kt) {
    const uint32_t k0 = kt * kGemmBK;
    const unsigned char* p = base + (uint64_t)k0 * k_step;   // (uniform)
    if (k0 + kGemmBK > K) {   // the short last k tile: what lies past K is read where it ends with K
      uint32_t back[R];
      static_for<R>([&](auto i) {
        uint32_t row, k;
        unit((uint32_t)i, &row, &k);
        back[i] = gemm_any_back(LOAD, k0, k, K, k_step);
      });
      static_for<R>([&](auto i) { regs[i] = *reinterpret_cast<const u32x4_any*>(p + ((int64_t)off[i] - (int64_t)back[i])); });
    } else {
      static_for<R>([&](auto i) { regs[i] = *reinterpret_cast<const u32x4_any*>(p + off[i]); });
    }
  }
  // parks k tile kt, which was asked for last: at = where this wavefront's first KiB of the tile lies in LDS
  __device__ __forceinline__ void park(unsigned char* at, uint32_t kt) {
    const uint32_t k0 = kt * kGemmBK;
    u32x4* slot = reinterpret_cast<u32x4*>(at + (t & 63u) * 16u);
    if (k0 + kGemmBK > K || (LOAD == kLoadRAny && extent % 8u != 0u && row0 + BR > extent)) {   // (uniform) an end to be moved or zeroed
      static_for<R>([&](auto i) {
        uint32_t row, k, move;
        unit((uint32_t)i, &row, &k);
        if constexpr (LOAD == kLoadKAny) gemm_any_start(k0 + k, K, &move);
        else gemm_any_start(row0 + row, extent, &move);
        slot[(int)i * 64] = select_or_zero(k0 + k < K, move_down_b16(regs[i], move));
      });
    } else {
      static_for<R>([&](auto i) { slot[(int)i * 64] = regs[i]; });
    }
  }
};

// The same tile for operands without vectors (or with vectors over a k mode of several short leaves), through registers.  Every
// load is an element (or a vector) at a 32-bit offset from the operand: the lanes' own part in a vector register, the part
// all lanes share in a scalar one.  One lane evaluates the k mode for one k of the tile; the others' offsets are read from it.
// k past K, and rows past the operand's extent, present an offset outside the buffer's range: zeros arrive (elements with the lanes along k
// repeat the last row instead: products nobody looks at).
// What bounds it: the vector memory path takes 64 addresses per instruction whatever their size, so an element costs what a
// vector costs; the lanes run along the mode whose neighbours share lines, and the eight elements a lane packs along the other.
// Measured on MI355X (bf16, us; element loads of 128 x 128 tiles -> this): no contiguous mode, 162 x 114 x 972 174 -> 10, 1024^3 183 -> 25,
// 4096^2 x 1024 524 -> 222; filters stored K,C,R,S, 64 x 115200 x 576 184 -> 43, 256 x 115200 x 1152 522 -> 244.
template <int BR, int LOAD, int WAVES>
struct GatherTileLoader {
  static constexpr int R = BR / 8 / WAVES;
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t K, t;
  bool vectors;          // (uniform)
  uint32_t off[R];       // bytes; elements along k: off[0] is the offset of row 8 R wave + lane, for the others to read
  uint32_t raw[8 * R];   // elements one a register; vectors four registers each

  __device__ __forceinline__ void init(const uint16_t* p, const GemmMode& rmode, uint32_t first_row, uint32_t rows, uint32_t Ktot, uint32_t lane,
                                       int32_t direct) {
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p), 0, 0xFFFFFFFFu, 0x00020000);
    K = Ktot;
    t = lane;
    vectors = gemm_gather_vectors(direct);
    if (LOAD == kLoadRGather && !vectors) {
      const uint32_t r = first_row + (t >> 6) * (R * 8u) + (t & 63u);   // (rows that do not exist: products nobody looks at)
      off[0] = 2u * gemm_mode_eval(rmode, r < rows ? r : rows - 1u);
      asm volatile("");   // (see fetch)
      return;
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
      uint32_t row, k;
      gemm_gather_unit(LOAD, vectors, BR, R, t, (uint32_t)i, &row, &k);
      const uint32_t r = first_row + row;
      off[i] = r < rows ? 2u * gemm_mode_eval(rmode, r) : 0xFFFFFFFFu;
    }
  }
  // asks for k tile kt
  __device__ __forceinline__ void fetch(uint32_t kt, const GemmMode& kmode) {
    const uint32_t k0 = kt * kGemmBK, lane = t & 63u;
    if (vectors) {
      // lane l stands for k vector l % 8, or for k l, of the tile
      const uint32_t kl = k0 + (LOAD == kLoadKGather ? 8u * (lane & 7u) : lane);
      const uint32_t k_off = 2u * gemm_mode_eval(kmode, kl < K ? kl : 0u);
      static_for<R>([&](auto i) {
        uint32_t row, k;
        gemm_gather_unit(LOAD, true, BR, R, t, (uint32_t)i, &row, &k);
        const uint32_t theirs = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(4u * (LOAD == kLoadKGather ? k / 8u : k)), (int)k_off);
        const uint32_t at = off[i] != 0xFFFFFFFFu && k0 + k < K ? off[i] + theirs : 0xFFFFFFFFu;
        const u32x4 v = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)at, 0, 0));
        static_for<4>([&](auto d) { raw[4 * i + d] = v[(int)d]; });
      });
      asm volatile("");   // (keeps the compiler from merging the two branches' last stores to `raw` into one at a variable index, which would put it in memory)
      return;
    }
    const uint32_t k_off = k0 + lane < K ? 2u * gemm_mode_eval(kmode, k0 + lane) : 0xFFFFFFFFu;   // of k k0 + lane
    static_for<R>([&](auto i) {
      static_for<8>([&](auto j) {
        uint32_t at, shared = 0u;   // the lane's part, the part of all lanes
        if constexpr (LOAD == kLoadRGather) {
          at = k_off;
          shared = (uint32_t)__builtin_amdgcn_readlane((int)off[0], 8 * i + j);
        } else {
          const uint32_t first = ((uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6)) * R + (uint32_t)i) * 64u / BR * 8u + (uint32_t)j;   // k inside the tile, of lane 0
          uint32_t its = (uint32_t)__builtin_amdgcn_readlane((int)k_off, (int)first);
          if constexpr (BR < 64) {
            const uint32_t upper = (uint32_t)__builtin_amdgcn_readlane((int)k_off, (int)first + 8);
            its = lane >= (uint32_t)BR ? upper : its;
            at = its != 0xFFFFFFFFu && off[i] != 0xFFFFFFFFu ? off[i] + its : 0xFFFFFFFFu;
          } else {
            at = its != 0xFFFFFFFFu ? off[i] : 0xFFFFFFFFu;
            shared = its != 0xFFFFFFFFu ? its : 0u;
          }
        }
        raw[8 * i + j] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rsrc, (int)at, (int)shared, 0);
      });
    });
  }
  // parks the k tile that was asked for last: at = where this wavefront's share of the tile lies in LDS
  __device__ __forceinline__ void park(unsigned char* at, uint32_t) {
    if (vectors) {
      u32x4* slot = reinterpret_cast<u32x4*>(at + (t & 63u) * 16u);
      static_for<R>([&](auto i) { slot[(int)i * 64] = u32x4{raw[4 * i], raw[4 * i + 1], raw[4 * i + 2], raw[4 * i + 3]}; });
      return;
    }
    unsigned char* tile = at - (t >> 6) * (R * 1024u);
    static_for<R>([&](auto i) {
      uint32_t row, k;
      gemm_gather_unit(LOAD, false, BR, R, t, (uint32_t)i, &row, &k);
      u32x4 v;
      static_for<4>([&](auto d) { v[(int)d] = raw[8 * i + 2 * d] | (raw[8 * i + 2 * d + 1] << 16); });
      *reinterpret_cast<u32x4*>(tile + (LOAD == kLoadKGather ? gemm_lds_offset(row, k / 8u) : gemm_rdirect_lds_offset(BR, k, row))) = v;
    });
  }
};
template <int BR, int LOAD, int WAVES>
using TileLoader = std::conditional_t<
    LOAD == kLoadKLeaves, LeavesTileLoader<BR, WAVES>,
    std::conditional_t<gemm_load_is_gather(LOAD), GatherTileLoader<BR, LOAD, WAVES>,
                       std::conditional_t<gemm_load_is_any(LOAD), AnyTileLoader<BR, LOAD, WAVES>, DirectTileLoader<BR, LOAD, WAVES>>>>;
// (which loads an operand without vectors takes is a matter of its plan, not of the kernel)
template <int LOAD, typename Loader>
__device__ __forceinline__ void init_loader(Loader& l, const uint16_t* p, const GemmMode& rmode, const GemmMode& kmode, uint32_t row0, uint32_t rows,
                                            uint32_t K, uint32_t lane, int32_t direct) {
  if constexpr (gemm_load_is_gather(LOAD)) l.init(p, rmode, row0, rows, K, lane, direct);
  else l.init(p, rmode, kmode, row0, rows, K, lane);
}
template <int LOAD, typename Loader>
__device__ __forceinline__ void fetch_tile(Loader& l, uint32_t kt, const GemmMode& kmode) {
  if constexpr (gemm_load_is_gather(LOAD)) l.fetch(kt, kmode);
  else l.fetch(kt);
}

// Fragment of rows row .. row + 31, k step kk of an operand's tile of BR rows at LDS address `tile`: this lane's 8 elements.
// (A tile of 16 rows stands twice in its fragment; the second half's products are never looked at.)
template <int BR, int LOAD, typename KK>
__device__ __forceinline__ u32x4 direct_fragment(const unsigned char* tile, uint32_t lane, uint32_t row, KK kk) {
  if constexpr (gemm_load_is_k_major(LOAD))
    return lds_read_tr_16x8<BR>(tile + gemm_rdirect_frag_offset(BR, lane, row, 8u * mfma_ab_kvec(lane)), kk);
  else
    return *reinterpret_cast<const u32x4*>(tile + gemm_lds_offset((row + mfma_ab_row(lane)) & (BR - 1u), 2u * (uint32_t)kk + mfma_ab_kvec(lane)));
}

// The units of a TM x TN tile of C that a lane of LANES adds sums to (gemm_sum_of): their old values are asked for ahead of
// time, the sums come out of LDS and go back in whole runs of C.
template <int TM, int TN, int LANES, bool C_VEC>
struct SumUnits {
  static constexpr int UNITS = TM * TN / 4, N = (UNITS + LANES - 1) / LANES;
  f32x4 old[N];
  uint32_t off[N][C_VEC ? 1 : 4];
  __device__ __forceinline__ void request(const GemmParams& P, const float* C, uint32_t m0, uint32_t n0, uint32_t tid) {
    static_for<N>([&](auto j) {
      uint32_t m4, n;
      gemm_sum_of(TM, TN, C_VEC, tid + (uint32_t)j * LANES, &m4, &n);
      const uint32_t m = m0 + 4u * m4;
      // units that do not exist read the last ones that do: no branch around the loads
      const uint32_t n_off = gemm_mode_eval(P.c_n, n0 + n < P.N ? n0 + n : P.N - 1u);
      if constexpr (C_VEC) {
        off[j][0] = gemm_mode_eval(P.c_m, m < P.M ? m : P.M - 4u) + n_off;
        old[j] = *reinterpret_cast<const f32x4*>(C + off[j][0]);
      } else {
        static_for<4>([&](auto v) {
          off[j][(int)v] = gemm_mode_eval(P.c_m, m + (uint32_t)v < P.M ? m + (uint32_t)v : P.M - 1u) + n_off;
          old[j][(int)v] = C[off[j][(int)v]];
        });
      }
    });
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);   // the operands' loads come after these
  }
  template <typename F>
  __device__ __forceinline__ void add(const GemmParams& P, float* C, uint32_t m0, uint32_t n0, uint32_t tid, F&& sum_of) {
    static_for<N>([&](auto j) {   // every sum first: a wait behind each would make a chain of LDS round trips
      uint32_t m4, n;
      gemm_sum_of(TM, TN, C_VEC, (tid + (uint32_t)j * LANES) % UNITS, &m4, &n);
      old[j] += sum_of(gemm_sum_unit(TM, TN, m4, n));
    });
    static_for<N>([&](auto j) {
      uint32_t m4, n;
      gemm_sum_of(TM, TN, C_VEC, tid + (uint32_t)j * LANES, &m4, &n);
      const uint32_t m = m0 + 4u * m4;
      const bool in = (UNITS % LANES == 0 || tid + (uint32_t)j * LANES < (uint32_t)UNITS) && n0 + n < P.N;
      if constexpr (C_VEC) {
        if (in && m < P.M) *reinterpret_cast<f32x4*>(C + off[j][0]) = old[j];
      } else {
        static_for<4>([&](auto v) {
          if (in && m + (uint32_t)v < P.M) C[off[j][(int)v]] = old[j][(int)v];
        });
      }
    });
  }
};

}  // namespace lc
