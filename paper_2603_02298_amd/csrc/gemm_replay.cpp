// Host walk of a GEMM plan (a checking device for tests, see gemm_plan.hpp): the kernel's loops over
// workgroups, lanes and k tiles with the same index functions (gemm_params.hpp), every global access
// checked against the buffers, the operand tiles passed through a byte model of LDS, and the matrix
// instruction replaced by its definition taken through the fragments' thread-value layouts.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "gemm_plan.hpp"

namespace lc {

namespace {

float bf16_to_float(uint16_t h) {
  uint32_t u = (uint32_t)h << 16;
  float f;
  std::memcpy(&f, &u, 4);
  return f;
}
float f16_to_float(uint16_t h) {
  const int sign = h >> 15, exp = (h >> 10) & 31, man = h & 1023;
  float v;
  if (exp == 0) v = std::ldexp((float)man, -24);
  else if (exp == 31) v = man ? NAN : INFINITY;
  else v = std::ldexp((float)(man + 1024), exp - 25);
  return sign ? -v : v;
}

struct Walker {
  const lc_gemm_plan& plan;
  const GemmParams& P;
  const uint16_t* A;
  const uint16_t* B;
  float* C;
  int64_t a_elems, b_elems, c_elems;
  bool ok = true;

  // loads one operand tile of k tile kt into the LDS model, lane by lane
  // lanes: how many load a tile together (a workgroup, or one wavefront of the split kernel); zero_rows: lanes past the
  // extent are answered with zeros instead of taking the last row
  void stage(const uint16_t* base, int64_t elems, const GemmMode& rmode, const GemmMode& kmode, int32_t load, uint32_t row0, uint32_t extent,
             uint32_t BR, uint32_t kt, unsigned char* tile, uint32_t lanes = (uint32_t)kBlock, bool zero_rows = false, int32_t direct = 0, uint32_t bk = (uint32_t)kGemmBK) {
    if (load == kLoadKDirect || load == kLoadKLeaves) {
      // every lane's 16 bytes land at byte 16 * lane of the 1 KiB its wavefront's instruction i fills
      const uint32_t rows_per_lane = BR * 8u / lanes;
      for (uint32_t tid = 0; tid < lanes; ++tid)
        for (uint32_t i = 0; i < rows_per_lane; ++i) {
          const uint32_t row = gemm_direct_row(rows_per_lane, tid, i), kv = gemm_direct_kvec(row, tid);
          const int64_t off = (int64_t)gemm_mode_eval(rmode, gemm_clamp_row(load, row0 + row, extent)) +
                              (load == kLoadKLeaves ? gemm_mode_eval(kmode, kt * kGemmBK + 8u * kv) : 8u * kv + gemm_mode_eval(kmode, kt * kGemmBK));
          const uint32_t lds_at = ((tid >> 6) * rows_per_lane + i) * 1024u + (tid & 63u) * 16u;
          if (lds_at != gemm_lds_offset(row, kv)) { ok = false; return; }
          if (kt * kGemmBK + 8u * kv >= P.K || (zero_rows && row0 + row >= extent)) {   // past K in a short last k tile: the lane's offset is out of range, zeros arrive
            std::memset(tile + lds_at, 0, 16);
            continue;
          }
          if (off % 8 != 0 || off + 8 > elems || kt * kGemmBK + 8u * kv + 8u > P.K) { ok = false; return; }
          for (uint32_t e = 1; e < 8; ++e)   // eight neighbours in memory
            if (gemm_mode_eval(kmode, kt * kGemmBK + 8u * kv + e) != gemm_mode_eval(kmode, kt * kGemmBK + 8u * kv) + e) { ok = false; return; }
          std::memcpy(tile + lds_at, base + off, 16);
        }
      return;
    }
    if (load == kLoadRDirect) {
      // k-major tile: lane l of instruction i of wavefront w fills 16-byte unit (w R + i) 64 + l
      const uint32_t rows_per_lane = BR * bk / 8u / lanes;   // (bk: 64, or pieces of 32 k rows)
      for (uint32_t tid = 0; tid < lanes; ++tid)
        for (uint32_t i = 0; i < rows_per_lane; ++i) {
          uint32_t k, row;
          gemm_rdirect_unit(BR, rows_per_lane, tid, i, &k, &row);
          const int64_t off = (int64_t)gemm_mode_eval(rmode, gemm_clamp_row(load, row0 + row, extent)) + (int64_t)k * kmode.lead_stride +
                              gemm_mode_eval(kmode, kt * bk);
          const uint32_t lds_at = ((tid >> 6) * rows_per_lane + i) * 1024u + (tid & 63u) * 16u;
          if (k >= bk || row + 8 > BR || lds_at != gemm_rdirect_lds_offset(BR, k, row)) { ok = false; return; }
          if (kt * bk + k >= P.K || (zero_rows && row0 + row >= extent)) {   // past K in a short last k tile: zeros arrive
            std::memset(tile + lds_at, 0, 16);
            continue;
          }
          // the k row's offset is what the k mode's layout function gives, and the slot is the one fragment reads expect
          if (off % 8 != 0 || off + 8 > elems ||
              (int64_t)k * kmode.lead_stride + gemm_mode_eval(kmode, kt * bk) != (int64_t)gemm_mode_eval(kmode, kt * bk + k)) {
            ok = false;
            return;
          }
          std::memcpy(tile + lds_at, base + off, 16);
        }
      return;
    }
    if (gemm_load_is_any(load)) {
      // the same units, read where they end with their mode when they would reach past it, and moved down
      const uint32_t R = BR * 8u / lanes;
      for (uint32_t tid = 0; tid < lanes; ++tid)
        for (uint32_t i = 0; i < R; ++i) {
          uint32_t k, row, move = 0, k_move = 0;
          if (load == kLoadKAny) {
            row = gemm_direct_row(R, tid, i);
            k = 8u * gemm_direct_kvec(row, tid);
          } else {
            gemm_rdirect_unit(BR, R, tid, i, &k, &row);
          }
          const uint32_t lds_at = ((tid >> 6) * R + i) * 1024u + (tid & 63u) * 16u, at_k = kt * kGemmBK + k;
          if (lds_at != (load == kLoadKAny ? gemm_lds_offset(row, k / 8u) : gemm_rdirect_lds_offset(BR, k, row))) { ok = false; return; }
          // the address as the lane forms it, in its own 32-bit steps; it has to be the place the two modes name
          const uint32_t k_step = 2u * kmode.lead_stride;
          const int64_t bytes = (int64_t)((uint64_t)(kt * kGemmBK) * k_step) + gemm_any_offset(load, rmode, row0 + row, extent, k, P.K, k_step) -
                                (int64_t)gemm_any_back(load, kt * kGemmBK, k, P.K, k_step);
          int64_t off;
          if (load == kLoadKAny) {
            off = (int64_t)gemm_mode_eval(rmode, row0 + row < extent ? row0 + row : extent - 1u) + gemm_any_start(at_k, P.K, &k_move);
          } else {
            const uint32_t from = gemm_any_start(row0 + row, extent, &move);
            off = (int64_t)gemm_mode_eval(rmode, from) + (int64_t)(at_k < P.K ? at_k : P.K - 1u) * kmode.lead_stride;
            for (uint32_t e = 0; e < 8; ++e)   // eight neighbours in memory
              if (gemm_mode_eval(rmode, from + e) != gemm_mode_eval(rmode, from) + e) { ok = false; return; }
          }
          if (bytes != 2 * off) { ok = false; return; }
          if (off < 0 || off + 8 > elems || move > 8u || k_move > 8u) { ok = false; return; }
          uint16_t v[8];
          std::memcpy(v, base + off, 16);
          for (uint32_t e = 0; e < 8; ++e) {
            const uint32_t from = e + move + k_move;
            const uint16_t x = from < 8u && at_k < P.K ? v[from] : 0;
            std::memcpy(tile + lds_at + 2u * e, &x, 2);
          }
        }
      return;
    }
    if (gemm_load_is_gather(load)) {
      // units of eight elements (or one vector) packed by their lane into the slot the fragment reads expect
      const uint32_t R = BR * 8u / lanes;
      for (uint32_t tid = 0; tid < lanes; ++tid)
        for (uint32_t i = 0; i < R; ++i) {
          uint32_t row, k;
          gemm_gather_unit(load, gemm_gather_vectors(direct), BR, R, tid, i, &row, &k);
          const uint32_t lds_at = load == kLoadKGather ? gemm_lds_offset(row, k / 8u) : gemm_rdirect_lds_offset(BR, k, row);
          if (row >= BR || k >= (uint32_t)kGemmBK || (load == kLoadKGather ? k % 8u : row % 8u) != 0) { ok = false; return; }
          if (gemm_gather_vectors(direct) && lds_at != ((tid >> 6) * R + i) * 1024u + (tid & 63u) * 16u) { ok = false; return; }
          for (uint32_t e = 0; e < 8; ++e) {
            const uint32_t at_row = row0 + row + (load == kLoadRGather ? e : 0u), at_k = kt * kGemmBK + k + (load == kLoadKGather ? e : 0u);
            uint16_t x = 0;
            if (at_k < P.K && (at_row < extent || (load == kLoadRGather && !gemm_gather_vectors(direct)))) {
              const int64_t off = (int64_t)gemm_mode_eval(rmode, at_row < extent ? at_row : extent - 1u) + gemm_mode_eval(kmode, at_k);
              if (off >= elems) { ok = false; return; }
              x = base[off];
              // a vector: eight neighbours in memory, all of them inside
              if (gemm_gather_vectors(direct)) {
                const int64_t first = (int64_t)gemm_mode_eval(rmode, row0 + row) + gemm_mode_eval(kmode, kt * kGemmBK + k);
                if (off != first + e || first % 8 != 0 || first + 8 > elems) { ok = false; return; }
              }
            } else if (gemm_gather_vectors(direct) && e > 0 && row0 + row < extent && kt * kGemmBK + k < P.K) { ok = false; return; }   // a vector straddles an end
            std::memcpy(tile + lds_at + 2u * e, &x, 2);
          }
        }
      return;
    }
    for (uint32_t tid = 0; tid < (uint32_t)kBlock; ++tid) {
      const uint32_t kv = gemm_lane_kvec(load, tid), k0 = kt * kGemmBK + kv * 8u;
      if (load == kLoadRVec) {
        if (tid >= BR) continue;
        const uint32_t block_row = gemm_lane_row(load, tid, 0);
        uint16_t blk[8][8] = {};   // [k][row]
        if (k0 < P.K) {
          const uint32_t rowoff = gemm_mode_eval(rmode, gemm_clamp_row(load, row0 + block_row, extent));
          const uint32_t koff = gemm_mode_eval(kmode, k0);
          for (uint32_t j = 0; j < 8; ++j) {
            const int64_t off = (int64_t)rowoff + koff + (int64_t)j * kmode.lead_stride;
            if (off % 8 != 0 || off + 8 > elems) { ok = false; return; }
            std::memcpy(blk[j], base + off, 16);
          }
        }
        for (uint32_t i = 0; i < 8; ++i) {
          uint16_t v[8];
          for (uint32_t j = 0; j < 8; ++j) v[j] = blk[j][i];
          std::memcpy(tile + gemm_lds_offset(block_row + i, kv), v, 16);
        }
      } else {
        for (uint32_t i = 0; i < BR / 32; ++i) {
          const uint32_t row = gemm_lane_row(load, tid, i);
          const uint32_t rowoff = gemm_mode_eval(rmode, gemm_clamp_row(load, row0 + row, extent));
          uint16_t v[8] = {};
          if (load == kLoadKVec) {
            if (k0 < P.K) {
              const int64_t off = (int64_t)rowoff + gemm_mode_eval(kmode, k0);
              if (off % 8 != 0 || off + 8 > elems) { ok = false; return; }
              std::memcpy(v, base + off, 16);
            }
          } else {
            for (uint32_t j = 0; j < 8; ++j)
              if (k0 + j < P.K) {
                const int64_t off = (int64_t)rowoff + gemm_mode_eval(kmode, k0 + j);
                if (off >= elems) { ok = false; return; }
                v[j] = base[off];
              }
          }
          std::memcpy(tile + gemm_lds_offset(row, kv), v, 16);
        }
      }
    }
  }

  // What a wavefront's lanes receive for one 32 x 16 fragment (rows row_base .. + 31 of the operand tile, k step kk):
  // out[lane][v], v < 8.  Row-major tiles: one 16-byte read per lane.  k-major tiles: two LDS transpose loads
  // (ds_read_b64_tr_b16), whose definition is applied here to the addresses the lanes present: within each group of
  // 16 lanes, lane i's element e is element i % 4 of the 8 bytes lane 4 e + i / 4 points at.
  void fragment(const unsigned char* tile, int32_t load, uint32_t BR, uint32_t row_base, uint32_t kk, uint16_t (*out)[8]) {
    for (uint32_t lane = 0; lane < 64; ++lane) {
      if (!gemm_load_is_k_major(load)) {
        std::memcpy(out[lane], tile + gemm_lds_offset((row_base + mfma_ab_row(lane)) % BR, 2u * kk + mfma_ab_kvec(lane)), 16);
        continue;
      }
      for (uint32_t h = 0; h < 2; ++h)
        for (uint32_t e = 0; e < 4; ++e) {
          const uint32_t src_lane = (lane & ~15u) + 4u * e + (lane & 15u) / 4u;
          const uint32_t at = gemm_rdirect_frag_offset(BR, src_lane, row_base, 16u * kk + 8u * mfma_ab_kvec(src_lane) + 4u * h);
          if (at % 8 != 0 || at + 8 > BR * 128u) { ok = false; return; }
          std::memcpy(&out[lane][4 * h + e], tile + at + 2u * (lane & 3u), 2);
        }
    }
  }
};

// one 32 x 32 fragment product of k step kk, added to a TM x TN accumulator at (row, col)
struct FragmentProduct {
  Layout tv_a, tv_b, tv_c;
  float (*to_float)(uint16_t);
  bool run(Walker& w, const unsigned char* a_tile, int32_t a_kind, uint32_t BM, uint32_t row, const unsigned char* b_tile, int32_t b_kind,
           uint32_t BN, uint32_t col, uint32_t kk, float* acc) {
    // gather the two 32 x 16 fragments from the lanes' LDS reads, through the thread-value layouts
    float fa[32][16], fb[32][16];
    uint16_t va[64][8], vb[64][8];
    w.fragment(a_tile, a_kind, BM, row, kk, va);
    w.fragment(b_tile, b_kind, BN, col, kk, vb);
    if (!w.ok) return false;
    for (uint32_t lane = 0; lane < 64; ++lane)
      for (uint32_t v = 0; v < 8; ++v) {
        const int64_t ca = tv_a((int64_t)lane + 64 * v), cb = tv_b((int64_t)lane + 64 * v);   // row + 32 k
        fa[ca % 32][ca / 32] = to_float(va[lane][v]);
        fb[cb % 32][cb / 32] = to_float(vb[lane][v]);
      }
    // D = A B^T + D, then back to the lanes' accumulators through the C fragment layout
    for (uint32_t lane = 0; lane < 64; ++lane)
      for (uint32_t v = 0; v < 16; ++v) {
        const int64_t cc = tv_c((int64_t)lane + 64 * v);   // m + 32 n
        const uint32_t r = (uint32_t)(cc % 32), c = (uint32_t)(cc / 32);
        if (r != mfma_c_row(lane, v) || c != mfma_c_col(lane)) return false;
        float sum = 0.f;
        if (col + c >= BN) continue;   // a tile of 16 columns stands twice in its fragment
        for (uint32_t k = 0; k < 16; ++k) sum += fa[r][k] * fb[c][k];
        acc[(size_t)(row + r) * BN + (col + c)] += sum;
      }
    return true;
  }
};

// The split kernel: every wavefront's k tiles into a partial tile of its own, the partials into units of LDS, the units
// summed in the order of the wavefronts and added to C.  The stream kernel: one tile, loaded by four wavefronts that hold
// a quarter of its sums each, through the same units.
lc_status_t replay_sums(const lc_gemm_plan& plan, Walker& w, FragmentProduct& product, float* c_all, int64_t c_all_elems) {
  const GemmParams& P = w.P;
  const uint32_t TM = (uint32_t)plan.tile_m, TN = (uint32_t)plan.tile_n, units = TM * TN / 4u;
  const bool split = plan.split_waves > 0;
  const uint32_t W = split ? (uint32_t)plan.split_waves : 1u, lanes = split ? 64u : (uint32_t)kBlock, QM = split ? TM : TM / 2u, QN = split ? TN : TN / 2u;
  const int32_t a_kind = gemm_effective_load(P.a_load, P.a_direct), b_kind = gemm_effective_load(P.b_load, P.b_direct);
  const bool pieces = !split && plan.stages == 4;   // k tiles of 32
  const uint32_t bk = pieces ? 32u : (uint32_t)kGemmBK, k_steps = pieces ? (P.K + 31u) / 32u : P.k_tiles;
  if (plan.stages < 1 || TM * TN * 4u > plan.lds_bytes || plan.lds_bytes != W * (unsigned)plan.stages * (TM + TN) * (pieces ? 64u : 128u) || (pieces && (a_kind != kLoadRDirect || b_kind != kLoadRDirect)) || !P.a_direct || !P.b_direct) return LC_ERR_INVALID_ARG;
  const uint32_t per_batch = P.tiles_m * P.tiles_n, n_tiles = per_batch * P.L;
  std::vector<unsigned char> lds((TM + TN) * 128u);
  std::vector<float> acc((size_t)TM * TN), parts((size_t)W * units * 4u);
  std::vector<char> covered(n_tiles, 0);
  const uint16_t *a_all = w.A, *b_all = w.B;
  const int64_t a_elems = w.a_elems, b_elems = w.b_elems;
  for (uint32_t block = 0; block < n_tiles; ++block) {
    const uint32_t order = gemm_tile_order_of_block(block, n_tiles);
    if (order >= n_tiles || covered[order]) return LC_ERR_INVALID_ARG;   // every tile exactly once
    covered[order] = 1;
    const uint32_t batch = order / per_batch;
    uint32_t tm, tn;
    gemm_tile_of_order(P, order - batch * per_batch, &tm, &tn);
    if (tm >= P.tiles_m || tn >= P.tiles_n) return LC_ERR_INVALID_ARG;
    const uint32_t m0 = tm * TM, n0 = tn * TN, ao = gemm_mode_eval(P.a_l, batch), bo = gemm_mode_eval(P.b_l, batch), co = gemm_mode_eval(P.c_l, batch);
    if (ao > a_elems || bo > b_elems || co > c_all_elems) return LC_ERR_INVALID_ARG;
    w.A = a_all + ao; w.a_elems = a_elems - ao;
    w.B = b_all + bo; w.b_elems = b_elems - bo;
    float* c = c_all + co;
    const int64_t c_elems = c_all_elems - co;
    for (uint32_t wave = 0; wave < W; ++wave) {
      std::fill(acc.begin(), acc.end(), 0.f);
      for (uint32_t kt = wave; kt < k_steps; kt += W) {
        w.stage(w.A, w.a_elems, P.a_r, P.a_k, a_kind, m0, P.M, TM, kt, lds.data(), lanes, true, P.a_direct, bk);
        w.stage(w.B, w.b_elems, P.b_r, P.b_k, b_kind, n0, P.N, TN, kt, lds.data() + TM * 128u, lanes, true, P.b_direct, bk);
        if (!w.ok) return LC_ERR_INVALID_ARG;
        for (uint32_t kk = 0; kk < bk / 16; ++kk)
          for (uint32_t i = 0; i < TM / 32; ++i)
            for (uint32_t j = 0; j < (TN + 31) / 32; ++j)
              if (!product.run(w, lds.data(), a_kind, TM, 32u * i, lds.data() + TM * 128u, b_kind, TN, 32u * j, kk, acc.data())) return LC_ERR_INVALID_ARG;
      }
      std::vector<char> written(units, 0);
      for (uint32_t tid = 0; tid < lanes; ++tid)
        for (uint32_t i = 0; i < QM / 32; ++i)
          for (uint32_t j = 0; j < (QN + 31) / 32; ++j)
            for (uint32_t g = 0; g < 4; ++g) {
              const uint32_t lane = tid & 63u, wm = (tid >> 6) & 1u, wn = tid >> 7;
              const uint32_t row = wm * QM + 32u * i + mfma_c_row(lane, 4u * g), col = wn * QN + 32u * j + mfma_c_col(lane), unit = gemm_sum_unit(TM, TN, row / 4u, col);
              if (col >= TN) continue;
              if (row % 4u != 0 || unit >= units || written[unit]) return LC_ERR_INVALID_ARG;
              written[unit] = 1;
              for (uint32_t v = 0; v < 4; ++v) parts[((size_t)wave * units + unit) * 4u + v] = acc[(size_t)(row + v) * TN + col];
            }
    }
    std::vector<char> added(units, 0);
    for (uint32_t u = 0; u < units; ++u) {
      uint32_t m4, nl;
      gemm_sum_of(TM, TN, P.c_vec, u, &m4, &nl);
      const uint32_t unit = gemm_sum_unit(TM, TN, m4, nl), m = m0 + 4u * m4, n = n0 + nl;
      if (m4 >= TM / 4u || nl >= TN || unit >= units || added[unit]) return LC_ERR_INVALID_ARG;
      added[unit] = 1;
      for (uint32_t v = 0; v < 4; ++v) {
        if (n >= P.N || m + v >= P.M) continue;
        const int64_t off = (int64_t)gemm_mode_eval(P.c_m, m + v) + gemm_mode_eval(P.c_n, n);
        if (off >= c_elems) return LC_ERR_INVALID_ARG;
        // one 16-byte access per unit: the four rows are there and follow each other from an aligned place
        if (P.c_vec && (m + 4u > P.M || off != (int64_t)gemm_mode_eval(P.c_m, m) + gemm_mode_eval(P.c_n, n) + v || (off - v) % 4 != 0)) return LC_ERR_INVALID_ARG;
        float sum = 0.f;
        for (uint32_t wave = 0; wave < W; ++wave) sum += parts[((size_t)wave * units + unit) * 4u + v];
        c[off] += sum;
      }
    }
  }
  return LC_OK;
}

}  // namespace

lc_status_t gemm_replay_on_host(const lc_gemm_plan& plan, const uint16_t* a, int64_t a_elems, const uint16_t* b, int64_t b_elems, float* c,
                                int64_t c_elems) {
  if (!a || !b || !c) return LC_ERR_INVALID_ARG;
  if (a_elems < plan.a_cosize || b_elems < plan.b_cosize || c_elems < plan.c_cosize) return LC_ERR_INVALID_ARG;
  const GemmParams& P = plan.params;
  Walker w{plan, P, plan.exchanged ? b : a, plan.exchanged ? a : b, c, plan.exchanged ? b_elems : a_elems,
           plan.exchanged ? a_elems : b_elems, c_elems};
  FragmentProduct product;
  mfma_fragment_layout(0, &product.tv_a);
  mfma_fragment_layout(1, &product.tv_b);
  mfma_fragment_layout(2, &product.tv_c);
  product.to_float = plan.ab_dtype == LC_BF16 ? bf16_to_float : f16_to_float;
  if (plan.stages > 0) return replay_sums(plan, w, product, c, c_elems);
  const uint32_t BM = (uint32_t)plan.tile_m, BN = (uint32_t)plan.tile_n, WMB = BM / 64, WNB = BN / 64;
  if (plan.lds_bytes != (P.a_direct ? 5u * std::max(BM, BN) * 128u : 2u * (BM + BN) * 128u)) return LC_ERR_INVALID_ARG;
  std::vector<unsigned char> lds((BM + BN) * 128u);   // one k tile of A and B is enough for a sequential walk
  std::vector<float> acc((size_t)BM * BN);
  std::vector<char> covered((size_t)P.tiles_m * P.tiles_n, 0);
  const uint32_t n_tiles = P.tiles_m * P.tiles_n;
  const int32_t a_kind = gemm_effective_load(P.a_load, P.a_direct), b_kind = gemm_effective_load(P.b_load, P.b_direct);
  const uint16_t* const a_all = w.A;
  const uint16_t* const b_all = w.B;
  float* const c_all = c;
  const int64_t a_all_elems = w.a_elems, b_all_elems = w.b_elems, c_all_elems = c_elems;
  for (uint32_t batch = 0; batch < P.L; ++batch) {
  // the batch entry's offsets are folded into the three base pointers, as the kernel does with blockIdx.y
  const uint32_t ao = gemm_mode_eval(P.a_l, batch), bo = gemm_mode_eval(P.b_l, batch), co = gemm_mode_eval(P.c_l, batch);
  if (ao > a_all_elems || bo > b_all_elems || co > c_all_elems) return LC_ERR_INVALID_ARG;
  w.A = a_all + ao;
  w.B = b_all + bo;
  w.a_elems = a_all_elems - ao;
  w.b_elems = b_all_elems - bo;
  c = c_all + co;
  c_elems = c_all_elems - co;
  std::fill(covered.begin(), covered.end(), 0);
  for (uint32_t block = 0; block < n_tiles; ++block) {
    uint32_t tm, tn;
    const uint32_t order = gemm_tile_order_of_block(block, n_tiles);
    if (order >= n_tiles) return LC_ERR_INVALID_ARG;
    gemm_tile_of_order(P, order, &tm, &tn);
    if (tm >= P.tiles_m || tn >= P.tiles_n || covered[(size_t)tm * P.tiles_n + tn]) return LC_ERR_INVALID_ARG;   // every tile exactly once
    covered[(size_t)tm * P.tiles_n + tn] = 1;
    const uint32_t m0 = tm * BM, n0 = tn * BN;
    std::fill(acc.begin(), acc.end(), 0.f);
    for (uint32_t kt = 0; kt < P.k_tiles; ++kt) {
      w.stage(w.A, w.a_elems, P.a_r, P.a_k, a_kind, m0, P.M, BM, kt, lds.data());
      w.stage(w.B, w.b_elems, P.b_r, P.b_k, b_kind, n0, P.N, BN, kt, lds.data() + BM * 128u);
      if (!w.ok) return LC_ERR_INVALID_ARG;
      for (uint32_t wave = 0; wave < 4; ++wave) {
        const uint32_t wm = wave & 1u, wn = wave >> 1;
        for (uint32_t kk = 0; kk < kGemmBK / 16; ++kk)
          for (uint32_t i = 0; i < WMB; ++i)
            for (uint32_t j = 0; j < WNB; ++j)
              if (!product.run(w, lds.data(), a_kind, BM, wm * WMB * 32u + 32u * i, lds.data() + BM * 128u, b_kind, BN, wn * WNB * 32u + 32u * j, kk,
                               acc.data()))
                return LC_ERR_INVALID_ARG;
      }
    }
    // epilogue, lane by lane
    for (uint32_t tid = 0; tid < (uint32_t)kBlock; ++tid) {
      const uint32_t lane = tid & 63u, wave = tid >> 6, wm = wave & 1u, wn = wave >> 1;
      for (uint32_t j = 0; j < WNB; ++j) {
        const uint32_t nl = wn * WNB * 32u + 32u * j + mfma_c_col(lane), n = n0 + nl;
        if (n >= P.N) continue;
        const uint32_t noff = gemm_mode_eval(P.c_n, n);
        for (uint32_t i = 0; i < WMB; ++i)
          for (uint32_t g = 0; g < 4; ++g) {
            const uint32_t ml = wm * WMB * 32u + 32u * i + mfma_c_row(lane, 4u * g), m = m0 + ml;
            if (P.c_vec) {
              if (m >= P.M) continue;
              const int64_t off = (int64_t)gemm_mode_eval(P.c_m, m) + noff;
              if (off % 4 != 0 || off + 4 > c_elems || m + 4 > P.M) return LC_ERR_INVALID_ARG;
              for (uint32_t v = 0; v < 4; ++v) c[off + v] += acc[(size_t)(ml + v) * BN + nl];
            } else {
              for (uint32_t v = 0; v < 4; ++v)
                if (m + v < P.M) {
                  const int64_t off = (int64_t)gemm_mode_eval(P.c_m, m + v) + noff;
                  if (off >= c_elems) return LC_ERR_INVALID_ARG;
                  c[off] += acc[(size_t)(ml + v) * BN + nl];
                }
            }
          }
      }
    }
  }
  }
  return LC_OK;
}

}  // namespace lc
