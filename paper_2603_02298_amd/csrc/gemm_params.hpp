// Kernel arguments and index arithmetic of the generic GEMM (Sec. 2.6.2 of "CuTe Layout Representation
// and Algebra"): C(m,n) += A(m,k) * B(n,k) for tensors given by rank-2 layouts.  A rank-2 layout is
// the sum of the layout functions of its two modes, L(r,k) = L_0(r) + L_1(k) (Eq. innerprod over the
// concatenation, Eq. concat), so each operand travels as two coalesced modes.  The functions here are
// shared by the device kernel and by the host walk that checks a plan's addresses without a GPU.
#pragma once
#include "kernel_params.hpp"

namespace lc {

constexpr int kGemmMaxLeaves = 4;   // leaves of one coalesced top-level mode
constexpr int kGemmBK = 64;         // k extent of a tile: 8 vectors of 8 sixteen-bit elements = one 128-byte LDS row

// how an operand tile is brought from global memory into LDS
enum GemmLoad : int32_t {
  kLoadKVec = 0,   // 16-byte vectors along k (k-mode leads with a stride-1 leaf): straight into place
  kLoadRVec = 1,   // 16-byte vectors along the row mode (m or n): 8x8 blocks transposed in registers
  kLoadElem = 2,   // element by element: any layout, any extent
  // kLoadKVec without the registers: 16-byte vectors along k sent by the memory pipeline straight into LDS.  Needs k tiles
  // that are contiguous along k (whole tiles inside the k mode's first leaf; a k mode of one leaf may end in a short tile,
  // whose lanes past K are answered with zeros); chosen at launch, a plan still says kLoadKVec.
  kLoadKDirect = 3,
  // kLoadRVec without the registers: the tile goes into LDS as it lies in memory (k rows of BR contiguous elements) and the
  // fragments are read with the LDS transpose load (ds_read_b64_tr_b16).  Same conditions; a plan still says kLoadRVec.
  kLoadRDirect = 4,
  // Vectors at any alignment, for operands with a contiguous mode whose rows do not start on 16-byte boundaries (odd sizes,
  // offset pointers): 16-byte loads from 2-byte-aligned addresses into registers, parked in the arrangement of kLoadKDirect
  // (along k) or kLoadRDirect (along the row mode).  Needs a k mode of one leaf; a plan still says kLoadElem.
  kLoadKAny = 5,
  kLoadRAny = 6,
  // Whatever neither of these takes, through registers into the arrangement of kLoadKDirect (kLoadKGather) or kLoadRDirect
  // (kLoadRGather): element by element with the lanes along the mode whose neighbours share more lines, or 16-byte vectors
  // whose k mode has leaves that k tiles are not whole in.  Any k mode; a plan still says what it found (gemm_gather_vectors).
  kLoadKGather = 7,
  kLoadRGather = 8,
  // kLoadKDirect over a k mode of leaves that k tiles are not whole in (a convolution's channels, where there are few): every
  // lane adds the offset of its own k vector.  The first leaf holds whole vectors; a plan still says kLoadKVec.
  kLoadKLeaves = 9
};
LC_HD constexpr bool gemm_load_is_any(int32_t load) { return load == kLoadKAny || load == kLoadRAny; }
LC_HD constexpr bool gemm_load_is_gather(int32_t load) { return load == kLoadKGather || load == kLoadRGather; }
LC_HD constexpr bool gemm_load_in_registers(int32_t load) { return gemm_load_is_any(load) || gemm_load_is_gather(load); }
LC_HD constexpr bool gemm_load_is_k_major(int32_t load) { return load == kLoadRDirect || load == kLoadRAny || load == kLoadRGather; }

// One coalesced mode: integral coordinate -> offset in elements (all offsets of a GEMM operand fit 31 bits).
// The leaves but the last are reduced modulo their extents, the last one takes what is left (Eq. idx2crd).
// Storage is branch-free for the kernel: the reduced leaves sit in front, padded with extent-1 leaves
// (quotient passes through, remainder 0), and the last leaf's stride always sits in last_stride.
struct GemmMode {
  int32_t n;                              // leaves of the coalesced mode (1 .. kGemmMaxLeaves)
  FastDiv div[kGemmMaxLeaves - 1];
  uint32_t stride[kGemmMaxLeaves - 1];
  uint32_t last_stride;
  uint32_t lead_stride;                   // stride of the first leaf (one step of the coordinate while it stays inside that leaf)
};
LC_HD uint32_t gemm_mode_eval(const GemmMode& g, uint32_t i) {
  uint32_t off = 0;
#pragma unroll
  for (int k = 0; k < kGemmMaxLeaves - 1; ++k) {
    uint32_t q, r;
    fd_divmod(i, g.div[k], &q, &r);
    off += r * g.stride[k];
    i = q;
  }
  return off + i * g.last_stride;
}

struct GemmParams {
  GemmMode a_r, a_k, b_r, b_k, c_m, c_n;   // A over (M,K), B over (N,K), C over (M,N)
  GemmMode a_l, b_l, c_l;                  // batch modes of the rank-3 form (Sec. 1): "1:0" for plain matrices
  uint32_t M, N, K, L;
  uint32_t tiles_m, tiles_n, k_tiles;
  int32_t a_load, b_load;                  // GemmLoad
  int32_t a_direct, b_direct;              // 1: the operand goes straight into LDS (kLoadKVec -> kLoadKDirect, kLoadRVec -> kLoadRDirect);
                                           // 2, 3: vectors at any alignment along k, along the row mode (kLoadKAny, kLoadRAny)
                                           // 4, 5: element by element, lanes along the row mode, along k (kLoadKGather, kLoadRGather)
                                           // 6, 7: k vectors, row vectors over any k mode (kLoadKGather, kLoadRGather)
                                           // 8: k vectors straight into LDS over any k mode (kLoadKLeaves)
  int32_t c_vec;                           // 1: four consecutive m are contiguous and 16-byte aligned in C
  uint32_t group_m;                        // tile rows walked together before moving on along n
};

// the load the kernel runs for an operand the plan classified as `load`
LC_HD int32_t gemm_effective_load(int32_t load, int32_t direct) {
  if (!direct) return load;
  if (direct == 8) return (int32_t)kLoadKLeaves;
  if (direct >= 4) return direct % 2 == 0 ? (int32_t)kLoadKGather : (int32_t)kLoadRGather;
  if (direct >= 2) return direct == 2 ? (int32_t)kLoadKAny : (int32_t)kLoadRAny;
  return load == kLoadKVec ? (int32_t)kLoadKDirect : (load == kLoadRVec ? (int32_t)kLoadRDirect : load);
}

LC_HD bool gemm_gather_vectors(int32_t direct) { return direct == 6 || direct == 7; }

// ---------------------------------------------------------------------------------------------
// Workgroup -> tile.  Workgroups are handed to the 8 XCDs round-robin and every XCD has its own L2,
// so XCD x takes a contiguous stretch of the tile order; the order itself walks group_m tile rows
// together along n, which keeps the A rows and B rows of concurrently running tiles few.
// ---------------------------------------------------------------------------------------------
constexpr uint32_t kXcds = 8;
LC_HD uint32_t gemm_tile_order_of_block(uint32_t block, uint32_t n_tiles) {
  const uint32_t xcd = block % kXcds, slot = block / kXcds;
  const uint32_t base = n_tiles / kXcds, extra = n_tiles % kXcds;
  return xcd * base + (xcd < extra ? xcd : extra) + slot;
}
LC_HD void gemm_tile_of_order(const GemmParams& P, uint32_t t, uint32_t* tm, uint32_t* tn) {
  const uint32_t width = P.group_m * P.tiles_n;
  const uint32_t group = t / width, in = t % width;
  const uint32_t first = group * P.group_m;
  const uint32_t rows = (P.tiles_m - first) < P.group_m ? (P.tiles_m - first) : P.group_m;
  *tm = first + in % rows;
  *tn = in / rows;
}

// ---------------------------------------------------------------------------------------------
// Operand tile in LDS: BR rows (m or n) of kGemmBK elements, 128 bytes per row, eight 16-byte
// vectors per row.  Vector kv of row r sits at slot kv ^ r ^ (r >> 3) (low three bits): this is the
// XOR layout (Sec. 2.3.2) under which all three access patterns below touch 16 distinct 16-byte
// bank groups per 16 lanes: fragment reads (16 rows, one kv), k-vector writes (2 rows x 8 kv) and
// the writes of transposed 8x8 blocks (8 row groups x 2 kv, rows of opposite parity for odd kv).
// ---------------------------------------------------------------------------------------------
LC_HD uint32_t gemm_lds_offset(uint32_t row, uint32_t kv) { return row * 128u + (((kv ^ row ^ (row >> 3)) & 7u) << 4); }

// ---------------------------------------------------------------------------------------------
// Lane -> what it loads (256 lanes).
//   kLoadKVec / kLoadElem: k vector lane % 8 of rows lane / 8 + 32 i, i < BR / 32: a quarter wavefront
//                          (16 lanes, one pass of a 16-byte load) reads two rows of 128 contiguous bytes
//   kLoadRVec            : the 8x8 block of rows 8 b .. 8 b + 7, b = lane % 8 + 8 (lane / 64), and k vector
//                          (lane / 8) % 8 (lanes < BR only): a quarter wavefront reads, for each of its two k
//                          vectors, 128 contiguous bytes along the row mode
// Rows past the end of the mode are clamped to its last row (last 8-row group for kLoadRVec): the
// tile then holds a copy of valid data there, which only feeds entries of C that are never stored.
// k past K parks zeros.
// ---------------------------------------------------------------------------------------------
LC_HD uint32_t gemm_lane_kvec(int32_t load, uint32_t lane) { return load == kLoadRVec ? (lane >> 3) & 7u : lane & 7u; }
LC_HD uint32_t gemm_lane_row(int32_t load, uint32_t lane, uint32_t i) {
  return load == kLoadRVec ? ((lane & 7u) + 8u * (lane >> 6)) * 8u : (lane >> 3) + 32u * i;
}
// ---------------------------------------------------------------------------------------------
// kLoadRDirect: the operand tile in LDS is k-major: row k holds the BR elements (BR / 8 slots of 16 bytes) of that k,
// the 8-element group g of the row mode in slot g ^ 4 (k % 4).  A transpose load of 16 lanes reads 16 rows x 4 k
// (4 k rows x 32 bytes); with this XOR layout (Sec. 2.3.2) the two lane groups that share a pass (rows 0..15 and
// 16..31 of a fragment) and their 4 k rows touch 16 distinct 16-byte bank groups.
// ---------------------------------------------------------------------------------------------
// Narrower tiles hold several k rows per 256 bytes of banks: with 64 rows (8 slots per k) two k rows share them and the XOR
// only has to part k rows 2 apart; with 32 rows (4 slots per k) four k rows fill them and nothing is folded.
// (192 rows are 24 slots: k rows 1 apart lie half the banks apart, k rows 2 apart are parted by the XOR)
LC_HD uint32_t gemm_rdirect_fold(uint32_t BR, uint32_t k) { return BR == 192u ? 2u * (k & 2u) : BR >= 128u ? 4u * (k & 3u) : BR == 64u ? 2u * (k & 2u) : 0u; }
LC_HD uint32_t gemm_rdirect_lds_offset(uint32_t BR, uint32_t k, uint32_t row) { return k * (BR * 2u) + ((((row >> 3) ^ gemm_rdirect_fold(BR, k))) << 4) + (row & 7u) * 2u; }
// Instruction i of wavefront w fills 1 KiB = 64 slots; lane l's slot is unit (w R + i) 64 + l of the tile: its k row and
// the 8-row group it must ask memory for.
LC_HD void gemm_rdirect_unit(uint32_t BR, uint32_t rows_per_lane, uint32_t tid, uint32_t i, uint32_t* k, uint32_t* row) {
  const uint32_t unit = ((tid >> 6) * rows_per_lane + i) * 64u + (tid & 63u), slots = BR / 8u;
  *k = unit / slots;
  *row = ((unit % slots) ^ gemm_rdirect_fold(BR, *k)) * 8u;
}
// ds_read_b64_tr_b16 (checked on the GPU with an in-bounds probe): within each group of 16 lanes, result lane i element e
// is element i % 4 of the 8 bytes that lane 4 e + i / 4 of the group points at.  Lane j of a group therefore points at
// rows 4 (j % 4) .. + 3 of its group's 16 rows, at k step j / 4 of the 4: lane i then holds row i at k .. k + 3.
// Byte offset (inside the operand's tile) for fragment rows row_base .. row_base + 31, k = k_base .. k_base + 3:
LC_HD uint32_t gemm_rdirect_frag_offset(uint32_t BR, uint32_t lane, uint32_t row_base, uint32_t k_base) {
  const uint32_t j = lane & 15u;
  return gemm_rdirect_lds_offset(BR, k_base + (j >> 2), row_base + 16u * ((lane >> 4) & 1u) + 4u * (j & 3u));
}

// kLoadKDirect: instruction i of wavefront w fills the 1 KiB of LDS that holds rows 8 (w R + i) .. + 7 of the tile
// (R = BR / 32 instructions per lane of four wavefronts, BR / 8 of one); lane l lands at byte 16 l of it, i.e. row + l / 8, slot l % 8, and therefore
// asks for the k vector that lives in that slot: kv = slot ^ row ^ (row >> 3).
LC_HD uint32_t gemm_direct_row(uint32_t rows_per_lane, uint32_t tid, uint32_t i) { return ((tid >> 6) * rows_per_lane + i) * 8u + ((tid & 63u) >> 3); }
LC_HD uint32_t gemm_direct_kvec(uint32_t row, uint32_t tid) { return ((tid & 7u) ^ row ^ (row >> 3)) & 7u; }
// Vectors at any alignment: a vector that would reach past the end of its mode is read where it ends with the mode (both
// ends of it are then inside) and moved down by what it was read early; what moves in from above is zero.  A vector that
// starts past the end reads the last one (rows: feeds entries of C that are never stored; k: zeroed).
// at: first coordinate of the vector, extent: of the mode (8 or more) -> where to read it, and by how many elements to move it
LC_HD uint32_t gemm_any_start(uint32_t at, uint32_t extent, uint32_t* move) {
  const uint32_t last = extent - 8u, from = at < last ? at : last;
  *move = at < extent ? at - from : 0u;
  return from;
}
// Where a lane reads unit (row, k) of the k tile that starts at k0, in bytes from the operand's first element:
// k0 * k_step + offset - back.  The offset is worked out once per workgroup and stays inside the operand for every k of a
// k tile (with K below the k tile it is already the place the last vector, or the last k row, is read at), so it fits 32 bits
// however close to 2^31 elements the operand ends; back is zero but in the short last k tile.
// row: of the vector's first element in the whole mode; k: its k inside the k tile; k_step: bytes from one k to the next
LC_HD uint32_t gemm_any_offset(int32_t load, const GemmMode& rmode, uint32_t row, uint32_t extent, uint32_t k, uint32_t K, uint32_t k_step) {
  uint32_t move;
  if (load == kLoadKAny) return 2u * (gemm_mode_eval(rmode, row < extent ? row : extent - 1u) + (K < (uint32_t)kGemmBK ? gemm_any_start(k, K, &move) : k));
  return 2u * gemm_mode_eval(rmode, gemm_any_start(row, extent, &move)) + (k < K ? k : K - 1u) * k_step;
}
LC_HD uint32_t gemm_any_back(int32_t load, uint32_t k0, uint32_t k, uint32_t K, uint32_t k_step) {
  uint32_t move;
  if (k0 + kGemmBK <= K || K < (uint32_t)kGemmBK) return 0u;
  if (load == kLoadKAny) return 2u * (k0 + k - gemm_any_start(k0 + k, K, &move));
  return k0 + k < K ? 0u : (k0 + k - (K - 1u)) * k_step;
}
// kLoadKGather / kLoadRGather element by element: unit i of a lane is eight elements that it packs into one 16-byte slot.
// Lanes along the row mode (kLoadKGather): eight k of one row, 64 neighbouring lanes = 64 rows (32 rows at two k vectors for
// a tile of 32), so every load instruction runs along the rows.  Lanes along k (kLoadRGather): eight rows at one k, the 64
// lanes = the 64 k of the tile, so every load runs along k.  Vectors: the units of kLoadKDirect / kLoadRDirect.
// *row, *k: first row and first k of the unit inside the tile
LC_HD void gemm_gather_unit(int32_t load, bool vectors, uint32_t BR, uint32_t units_per_lane, uint32_t tid, uint32_t i, uint32_t* row, uint32_t* k) {
  if (vectors && load == kLoadKGather) {
    *row = gemm_direct_row(units_per_lane, tid, i);
    *k = 8u * gemm_direct_kvec(*row, tid);
  } else if (vectors) {
    gemm_rdirect_unit(BR, units_per_lane, tid, i, k, row);
  } else if (load == kLoadKGather) {
    const uint32_t slot = ((tid >> 6) * units_per_lane + i) * 64u + (tid & 63u);
    *row = slot % BR;
    *k = 8u * (slot / BR);
  } else {
    *row = 8u * ((tid >> 6) * units_per_lane + i);
    *k = tid & 63u;
  }
}
LC_HD uint32_t gemm_clamp_row(int32_t load, uint32_t row, uint32_t extent) {
  const uint32_t last = load == kLoadRVec || load == kLoadRDirect ? extent - 8u : extent - 1u;
  return row < last ? row : last;
}

// ---------------------------------------------------------------------------------------------
// Split kernel: a workgroup of W wavefronts owns a TM x TN tile of C and its wavefronts share out the k tiles (wavefront w
// takes k tiles w, w + W, ...).  Each wavefront keeps operand tiles of its own in LDS -- the arrangements above for one
// wavefront: instruction i fills KiB i of the tile -- and a partial tile of C in registers; the partials are summed
// through LDS in the order of the wavefronts.
// Sums on their way to C through LDS (this kernel's partial tiles, the stream kernel's finished ones): TM x TN floats as
// 16-byte units of four consecutive m; unit (m4, n) = four rows from 4 m4 of column n.  They are written as the matrix
// instruction leaves them (8 lanes: 8 columns, one m4) and read back 16 lanes along m4 first (C contiguous along m) or
// along n; the XOR keeps both free of bank conflicts: the 16 lanes of a read pass (4-lane groups 0,3,5,6 or 1,2,4,7 of
// 32 lanes) hold 4 columns x 8 m4 (TM = 32), 2 x 16 (TM = 64) or 1 x 32 (TM >= 128).
// ---------------------------------------------------------------------------------------------
LC_HD uint32_t gemm_sum_unit(uint32_t TM, uint32_t TN, uint32_t m4, uint32_t n) {
  const uint32_t far = TM == 32u ? 0u : TM == 64u ? 2u * ((m4 >> 3) & 1u) : (m4 >> 2) & 3u;
  return m4 * TN + (n ^ (4u * (m4 & 3u)) ^ far);
}
// Unit u of the TM TN / 4 a workgroup adds to C: consecutive u run along m where C holds four consecutive m in a vector,
// along n otherwise.
LC_HD void gemm_sum_of(uint32_t TM, uint32_t TN, int32_t c_vec, uint32_t u, uint32_t* m4, uint32_t* n) {
  *m4 = c_vec ? u % (TM / 4u) : u / TN;
  *n = c_vec ? u / (TM / 4u) : u % TN;
}

// ---------------------------------------------------------------------------------------------
// MFMA fragments of v_mfma_f32_32x32x16 (bf16 / f16), as thread-value layouts (Sec. 3.3.4):
//   A fragment (32 x 16): lane t holds A(t % 32, 8 (t / 32) + v), v < 8   -> ((32,2),8):((1,256),32) on m + 32 k
//   B fragment (32 x 16): lane t holds B(t % 32, 8 (t / 32) + v)          -> the same on n + 32 k
//   C fragment (32 x 32): lane t holds C(8 (v / 4) + 4 (t / 32) + v % 4, t % 32), v < 16
//                                                                          -> ((32,2),(4,4)):((32,4),(1,8)) on m + 32 n
// ---------------------------------------------------------------------------------------------
LC_HD uint32_t mfma_ab_row(uint32_t lane) { return lane & 31u; }
LC_HD uint32_t mfma_ab_kvec(uint32_t lane) { return lane >> 5; }            // which 8-element k vector of the 16
LC_HD uint32_t mfma_c_row(uint32_t lane, uint32_t v) { return 8u * (v >> 2) + 4u * (lane >> 5) + (v & 3u); }
LC_HD uint32_t mfma_c_col(uint32_t lane) { return lane & 31u; }

}  // namespace lc
