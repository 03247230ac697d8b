#include "gemm_plan.hpp"

#include <algorithm>
#include <cstdlib>

#include "plan.hpp"

namespace lc {

namespace {

// one top-level mode, coalesced (Sec. 3.2), as the kernel's argument
lc_status_t fill_mode(const Modes& m, GemmMode* out) {
  if (m.empty() || (int)m.size() > kGemmMaxLeaves) return LC_ERR_TOO_LARGE;
  out->n = (int32_t)m.size();
  for (const Mode& x : m)
    if (x.extent >= (int64_t(1) << 31) || x.stride >= (int64_t(1) << 31)) return LC_ERR_TOO_LARGE;
  for (int k = 0; k < kGemmMaxLeaves - 1; ++k) {
    const bool reduced = k + 1 < (int)m.size();
    out->div[k] = make_fastdiv(reduced ? (uint32_t)m[k].extent : 1u);
    out->stride[k] = reduced ? (uint32_t)m[k].stride : 0u;
  }
  out->last_stride = (uint32_t)m.back().stride;
  out->lead_stride = (uint32_t)m.front().stride;
  return LC_OK;
}

// Does the mode lead with a stride-1 leaf whose extent is a multiple of `vec`?  Then `vec` consecutive
// coordinates starting at a multiple of `vec` are consecutive in memory.
bool leads_contiguous(const Modes& m, int64_t vec) { return m[0].stride == 1 && m[0].extent % vec == 0; }
// every stride except that of the leading leaf of `lead` is a multiple of `vec` (alignment of every vector)
bool strides_aligned(const Modes& lead, const Modes& other, int64_t vec) {
  for (size_t k = 1; k < lead.size(); ++k)
    if (lead[k].stride % vec != 0) return false;
  for (const Mode& x : other)
    if (x.stride % vec != 0) return false;
  return true;
}

int classify_operand(const Modes& row, const Modes& k, const Modes& batch, unsigned align_bytes) {
  auto plus_batch = [&](Modes other) {
    other.insert(other.end(), batch.begin(), batch.end());
    return other;
  };
  if (align_bytes % 16 == 0) {
    if (leads_contiguous(k, 8) && strides_aligned(k, plus_batch(row), 8)) return kLoadKVec;
    // vectors along the row mode, eight of them (k .. k + 7) per block: k must step evenly inside a block
    if (leads_contiguous(row, 8) && strides_aligned(row, plus_batch(k), 8) && k[0].extent % 8 == 0) return kLoadRVec;
  }
  return kLoadElem;
}

std::string mode_text(const Modes& m) { return Layout::flat(m).str(); }

int env_int(const char* name, int dflt) {
  const char* v = std::getenv(name);
  return (v && *v) ? std::atoi(v) : dflt;
}

// How a pair of operands is brought in.
struct Loads {
  int a, b;                  // GemmLoad, what a plan says
  int a_direct, b_direct;    // see GemmParams
  int a_gather, b_gather;    // what they are for gathered operands
  bool direct, any, gather;  // both straight into LDS, both in vectors at any alignment, both gathered through registers
};

// lines of 128 bytes, of line_elems elements each, that the first 64 coordinates of a mode touch
int lines_of(const Modes& m, int line_elems) {
  int64_t size = 1;
  for (const Mode& x : m) size *= x.extent;
  std::vector<int64_t> lines;
  for (int64_t i = 0; i < std::min<int64_t>(size, 64); ++i) {
    int64_t at = 0, rest = i;
    for (const Mode& x : m) { at += rest % x.extent * x.stride; rest /= x.extent; }
    lines.push_back(at / line_elems);
  }
  std::sort(lines.begin(), lines.end());
  return (int)(std::unique(lines.begin(), lines.end()) - lines.begin());
}

Loads choose_loads(const Modes& a_r, const Modes& a_k, const Modes& a_l, unsigned a_align, const Modes& b_r, const Modes& b_k, const Modes& b_l,
                   unsigned b_align, int64_t K) {
  Loads l;
  l.a = classify_operand(a_r, a_k, a_l, a_align);
  l.b = classify_operand(b_r, b_k, b_l, b_align);
  const int force = env_int("LC_TUNE_GEMM_LOAD", -1);   // tests: force the element-wise loads
  const int a_own = l.a, b_own = l.b;
  // element loads are compiled for both operands together: one operand that needs them takes the other along
  if (force == kLoadElem || l.a == kLoadElem || l.b == kLoadElem) l.a = l.b = kLoadElem;
  // straight into LDS: k tiles that are contiguous along k
  // (for row vectors: each of the tile's 64 k rows one even step of the k mode's first leaf from the tile's first);
  // compiled for pairs of operands that both qualify
  // A k mode of a single leaf may end in a short k tile: the lanes whose piece lies past K are answered with zeros
  // (k vectors: K a multiple of 8, so that no vector straddles K).
  auto direct_ok = [&](int load, const Modes& k) {
    if (load == kLoadElem) return false;
    if (K % kGemmBK == 0 && k[0].extent % kGemmBK == 0) return true;
    return k.size() == 1 && (load == kLoadRVec || K % 8 == 0) && env_int("LC_TUNE_GEMM_KTAIL", 1) != 0;
  };
  const int direct_env = env_int("LC_TUNE_GEMM_DIRECT", 3);   // bit 0: k vectors, bit 1: row vectors
  auto direct_on = [&](int load) { return (direct_env & (load == kLoadKVec ? 1 : 2)) != 0; };
  l.direct = direct_ok(l.a, a_k) && direct_ok(l.b, b_k) && direct_on(l.a) && direct_on(l.b);
  l.a_direct = l.b_direct = l.direct ? 1 : 0;
  // Operands with a contiguous mode that vectors do not fit (odd sizes, offset pointers): 16-byte loads at any alignment, for
  // pairs that both have one.  Measured on MI355X (bf16), element by element -> this: 1001 x 2003 x 1537 (all odd) 211 -> 22 us,
  // 3500^3 (no multiple of 8) 891 -> 158 us, 301 x 401 x 501 30 -> 5.5 us.
  auto any_kind = [&](const Modes& row, const Modes& k) -> int32_t {
    if (k.size() != 1) return 0;
    if (k[0].stride == 1 && K >= 8) return 2;
    const bool whole = row[0].extent % 8 == 0 || (row.size() == 1 && row[0].extent >= 8);
    return row[0].stride == 1 && whole ? 3 : 0;
  };
  l.any = l.a == kLoadElem && force != kLoadElem && any_kind(a_r, a_k) != 0 && any_kind(b_r, b_k) != 0;
  if (l.any) {
    l.a_direct = any_kind(a_r, a_k);
    l.b_direct = any_kind(b_r, b_k);
  }
  // What is left -- no contiguous mode, a k mode of several leaves beside an unaligned one, vectors whose k mode has leaves
  // that k tiles are not whole in -- is gathered through registers, each operand in its own way (lanes along the mode whose 64
  // neighbours touch fewer lines), on the split and stream kernels: faster than the tile kernels' element and staged loads at
  // every size measured (figures beside the loaders).
  l.gather = !l.direct && !l.any && force != kLoadElem && direct_env == 3 && env_int("LC_TUNE_GEMM_KTAIL", 1) != 0;
  auto gather_kind = [&](int own, const Modes& row, const Modes& k) -> int32_t {
    if (own != kLoadElem) return own == kLoadKVec ? 6 : 7;
    return lines_of(row, 64) <= lines_of(k, 64) ? 4 : 5;
  };
  l.a_gather = gather_kind(a_own, a_r, a_k);
  l.b_gather = gather_kind(b_own, b_r, b_k);
  if (l.a_gather == 6 && l.b_gather == 6) l.a_gather = l.b_gather = 8;   // k vectors on both sides: straight into LDS
  return l;
}

}  // namespace

lc_status_t mfma_fragment_layout(int which, Layout* out) {
  if (which == 0 || which == 1) {
    *out = Layout::tuple({Layout::flat({{32, 1}, {2, 256}}), Layout::leaf(8, 32)});
    return LC_OK;
  }
  if (which == 2) {
    *out = Layout::tuple({Layout::flat({{32, 32}, {2, 4}}), Layout::flat({{4, 1}, {4, 8}})});
    return LC_OK;
  }
  return LC_ERR_INVALID_ARG;
}

lc_status_t make_gemm_plan(const Layout& A_in, const Layout& B_in, const Layout& C_in, int ab_dtype, unsigned a_align,
                           unsigned b_align, unsigned c_align, lc_gemm_plan* out) {
  if (ab_dtype != LC_BF16 && ab_dtype != LC_F16) return LC_ERR_UNSUPPORTED_DTYPE;
  for (const Layout* L : {&A_in, &B_in, &C_in}) {
    lc_status_t st = validate(*L);
    if (st != LC_OK) return st;
    // matrices: shapes of rank 2 (Sec. 2.6.2); or all three of rank 3: the batched form of Sec. 1
    if (L->is_leaf() || (L->rank() != 2 && L->rank() != 3) || L->rank() != A_in.rank()) return LC_ERR_INVALID_ARG;
  }
  // preconditions of Sec. 2.6.2
  const int64_t M = A_in.mode(0).size(), K = A_in.mode(1).size(), N = B_in.mode(0).size();
  if (M != C_in.mode(0).size() || N != C_in.mode(1).size() || K != B_in.mode(1).size()) return LC_ERR_SIZE_MISMATCH;
  const bool batched = A_in.rank() == 3;
  const int64_t Lb = batched ? A_in.mode(2).size() : 1;
  if (batched && (Lb != B_in.mode(2).size() || Lb != C_in.mode(2).size())) return LC_ERR_SIZE_MISMATCH;
  if (Lb > 65535) return LC_ERR_TOO_LARGE;   // the tile kernels' second grid dimension is the batch index
  lc_gemm_plan plan;
  plan.ab_dtype = ab_dtype;
  plan.M = M;
  plan.N = N;
  plan.K = K;
  plan.L = Lb;
  plan.a_cosize = A_in.cosize();
  plan.b_cosize = B_in.cosize();
  plan.c_cosize = C_in.cosize();
  const int64_t lim = int64_t(1) << 31;
  if (plan.a_cosize >= lim || plan.b_cosize >= lim || plan.c_cosize >= lim || M >= lim || N >= lim || K >= lim) return LC_ERR_TOO_LARGE;

  // every mode coalesced on its own (Sec. 3.2, by-mode): the kernel evaluates L(r,k) = L_0(r) + L_1(k)
  Modes a_r = coalesce_modes(A_in.mode(0).leaves), a_k = coalesce_modes(A_in.mode(1).leaves);
  Modes b_r = coalesce_modes(B_in.mode(0).leaves), b_k = coalesce_modes(B_in.mode(1).leaves);
  Modes c_m = coalesce_modes(C_in.mode(0).leaves), c_n = coalesce_modes(C_in.mode(1).leaves);
  const Modes unit = {{1, 0}};
  Modes a_l = batched ? coalesce_modes(A_in.mode(2).leaves) : unit, b_l = batched ? coalesce_modes(B_in.mode(2).leaves) : unit;
  Modes c_l = batched ? coalesce_modes(C_in.mode(2).leaves) : unit;

  // C must not alias: many lanes add into it concurrently
  {
    Modes all = c_m;
    all.insert(all.end(), c_n.begin(), c_n.end());
    all.insert(all.end(), c_l.begin(), c_l.end());
    if (M * N * Lb > 1 && !layout_is_injective(all, M * N * Lb)) return LC_ERR_DST_ALIASES;
  }

  // The MFMA result fragment holds four consecutive rows (m) per lane and column.  When C is
  // contiguous along n instead, the roles are exchanged: C^T(n,m) += B(n,k) A(m,k) is the same GEMM
  // with the operands swapped and C's modes exchanged (Table gemm, row "NTT").
  auto with_batch = [](Modes other, const Modes& batch) {
    other.insert(other.end(), batch.begin(), batch.end());
    return other;
  };
  auto c_vec_ok = [&](const Modes& lead, const Modes& other) {
    return c_align % 16 == 0 && leads_contiguous(lead, 4) && strides_aligned(lead, with_batch(other, c_l), 4);
  };
  bool exchange = !c_vec_ok(c_m, c_n) && c_vec_ok(c_n, c_m);
  Loads loads = choose_loads(a_r, a_k, a_l, a_align, b_r, b_k, b_l, b_align, K);
  const int t_env = env_int("LC_TUNE_GEMM_TILE", 0);
  const bool free_choice = t_env == 0;
  // Vectors on both sides have the tile kernels' staged loads to fall back on, and these are better on large problems.  Measured on
  // MI355X (bf16, us; staged, gathered or over leaves): row vectors on both sides 1024^3 27.6, 12.4; 2048^3 59, 55; 4096^2 x 1024 68, 74; 4096^3 166,
  // 216; beside k vectors 1024^3 21.8, 11.8; 2048^3 49.9, 57.6; 1000 x 8000 x 960 34.4, 37.0; k vectors over leaves 1024^3 20.9, 10.3;
  // 4096^2 x 1024 69.5, 62.2; 4096^3 177.4, 179.8; 8192^2 x 2048 434.7, 433.4.
  auto in_tiles = [&](int64_t side) { return (M + side - 1) / side * ((N + side - 1) / side) * Lb; };
  const bool staged_pays = loads.a_gather == 8 ? K >= 3000 && in_tiles(256) >= 256 : loads.a_gather >= 6 && loads.b_gather >= 6 && in_tiles(128) >= 256;
  const bool indirect = loads.gather && (free_choice ? !staged_pays && env_int("LC_TUNE_GEMM_GATHER", 1) != 0 : t_env != 128 && t_env != 256 && t_env != 1285 && t_env != 3216);
  const bool leaves = indirect && loads.a_gather == 8, gather = indirect && !leaves;
  if (indirect) {
    loads.a_direct = loads.a_gather;
    loads.b_direct = loads.b_gather;
  }
  // Without vectors of four m the lanes of the split and stream kernels' update run along n, element by element: the mode of C whose
  // neighbours share more lines goes there, whichever way the operands come in; not for a few columns of operands with thin tiles, which are worth
  // more, nor for a few contiguous rows, where it gains nothing (gathered 5 x 1500 x 700 8.8 -> 9.0, 56 x 3044 x 3008 27.5 -> 30.0, up to 128 rows 0.99 on
  // average; over leaves 2 x 1500 x 216 3.8 -> 4.0, from 17 rows on faster).  Measured on MI355X over 600 problems of more than 16 rows and columns,
  // the exchanged order's time over the other's: C contiguous along m direct 0.79 on average (0.32 at best), vectors at any alignment 0.84,
  // gathered 0.88 (2382 x 1376 x 27 29.2 -> 24.9 us), over leaves 0.73; the closer mode along m and none contiguous 0.82, 0.84, 0.89, 0.81; the closer mode
  // along n 1.04 to 1.30.  The tile kernels of staged and element loads measured slower that way round (2 x 5560 x 64 10.8 -> 15.2 us, a
  // convolution of 35 x 13500 x 288 16.8 -> 21.4).
  if (!c_vec_ok(c_m, c_n) && !c_vec_ok(c_n, c_m))
    exchange = (gather ? M > 64 || c_m[0].stride != 1 : leaves ? M > 16 : (loads.direct || loads.any) && N > 16) && lines_of(c_m, 32) < lines_of(c_n, 32);
  if (env_int("LC_TUNE_GEMM_EXCHANGE", -1) >= 0) exchange = env_int("LC_TUNE_GEMM_EXCHANGE", 0) != 0;
  if (exchange) {
    std::swap(a_r, b_r);
    std::swap(a_k, b_k);
    std::swap(a_l, b_l);
    std::swap(c_m, c_n);
    std::swap(loads.a, loads.b);
    std::swap(loads.a_direct, loads.b_direct);
  }
  plan.exchanged = exchange;
  const int64_t kM = exchange ? N : M, kN = exchange ? M : N;

  GemmParams& P = plan.params;
  lc_status_t st;
  if ((st = fill_mode(a_r, &P.a_r)) != LC_OK || (st = fill_mode(a_k, &P.a_k)) != LC_OK || (st = fill_mode(b_r, &P.b_r)) != LC_OK ||
      (st = fill_mode(b_k, &P.b_k)) != LC_OK || (st = fill_mode(c_m, &P.c_m)) != LC_OK || (st = fill_mode(c_n, &P.c_n)) != LC_OK ||
      (st = fill_mode(a_l, &P.a_l)) != LC_OK || (st = fill_mode(b_l, &P.b_l)) != LC_OK || (st = fill_mode(c_l, &P.c_l)) != LC_OK)
    return st;
  P.M = (uint32_t)kM;
  P.N = (uint32_t)kN;
  P.K = (uint32_t)K;
  P.L = (uint32_t)Lb;
  P.a_load = loads.a;
  P.b_load = loads.b;
  P.a_direct = loads.a_direct;
  P.b_direct = loads.b_direct;
  const bool direct = loads.direct, any = loads.any;
  P.c_vec = c_vec_ok(c_m, c_n) ? 1 : 0;
  if (env_int("LC_TUNE_GEMM_CVEC", 1) == 0) P.c_vec = 0;
  unsigned need_a = P.a_load == kLoadElem ? 2u : 16u, need_b = P.b_load == kLoadElem ? 2u : 16u;
  plan.a_align = exchange ? need_b : need_a;
  plan.b_align = exchange ? need_a : need_b;
  plan.c_align = P.c_vec ? 16u : 4u;

  // Tile.  Split kernel (operands straight into LDS or in vectors at any alignment): while tiles of 64 x 64 leave a CU at most one workgroup, and then the smallest of
  // its tiles that does: the k tiles of a workgroup's tile go to its wavefronts, more tiles only take LDS from each other.
  // Measured on MI355X (bf16, start = 128 x 128 tiles): 512^3 11.1 us; 32 x 32 tiles (256 of them) 4.3, 32 x 64 4.7, 64 x 64
  // 6.2.  16 x 8192 x 8192 78 us; 32 x 32 27.6, 64 x 64 36.  64 x 8192 x 8192 92 us; 32 x 32 (512 tiles) 42.8, 64 x 32 (256) 33.4.
  // 1024^3 17.6 us; 32 x 64 (512 tiles) 10.8, 64 x 64 (256) 8.3.
  auto tiles_of = [&](int64_t tm, int64_t tn) { return (kM + tm - 1) / tm * ((kN + tn - 1) / tn) * Lb; };
  // LC_TUNE_GEMM_TILE: 256, 256192 (256 x 192), 192256, 128 (gathered operands: 1282), 12864 (128 x 64), 64128, 1285 (the ring of five 128 x 128 tiles); split kernel: 32, 64, 3216 (32 x 16), 3264 (32 x 64), 6432; 6464: the
  // stream kernel's 64 x 64
  auto take = [&](int tm, int tn, int waves, int stages) { plan.tile_m = tm; plan.tile_n = tn; plan.split_waves = waves; plan.stages = stages; };
  const bool thin = kN <= 16 && !indirect && (P.b_load == kLoadKVec || P.b_direct == 2), vectors = direct || any || indirect;
  const bool regs = any || gather;   // through registers: one pair of tiles
  // Gathered operands: an element costs the vector memory path what a vector costs, so a side of elements weighs eight times a side
  // of vectors, and tiles reach further along the vectors' side.
  const bool a_elem = gather && P.a_direct < 6, b_elem = gather && P.b_direct < 6, mixed = a_elem != b_elem;
  if (mixed && free_choice && tiles_of(32, 32) > 256) {
    // Measured on MI355X (bf16, us; filters stored K,C,R,S as elements, the activation in vectors; 32 x 64 split, 64 x 64, 128 x 64, 64 x 128, 128 x 128):
    // convolutions of 128 x 7128 x 144 6.9, 7.4, 10.2, 8.7, 12.2; 40 x 12696 x 1152 18.9, 29.6, 40.5, 33.1, 45.6; 64 x 17600 x 144 10.0, 8.8, 14.3, 8.9, 12.2;
    // 256 x 115200 x 1152 423, 360, 353, 244, 256; 64 x 115200 x 576 66, 56, 99, 43, 72; 256 x 25088 x 1152 96, 92, 103, 73, 71.
    if (a_elem ? tiles_of(32, 64) <= 512 : tiles_of(64, 32) <= 512) take(a_elem ? 32 : 64, a_elem ? 64 : 32, 4, 1);
    else take(a_elem ? 64 : 128, a_elem ? 128 : 64, 0, 2);
  } else if (vectors && (t_env == 3216 || free_choice) && thin && (!free_choice || tiles_of(32, 16) <= 256)) take(32, 16, 8, regs ? 1 : 3);
  else if (vectors && (t_env == 32 || (free_choice && tiles_of(32, 32) <= 256))) take(32, 32, 8, regs ? 1 : 2);
  // Short k loops leave the split kernel's wavefronts nothing to share: 64 x 64 tiles of the stream kernel are fewer and start with
  // less.  Measured on MI355X (us; split kernel's choice, then these): 736 x 680 x 128 4.94, 3.98; 632 x 952 x 120 5.45, 4.26;
  // 1008 x 472 x 112 (64 x 32) 4.58, 3.96; 800 x 352 x 184 (64 x 32) 3.97, 4.00; 64 x 64 tiles of 544 x 904 x 352 6.33, 5.56,
  // of 848 x 968 x 768 8.35, 9.23; with a single k tile 250 problems 0.81 of the time, 0.95 at worst.
  else if (free_choice && (direct || leaves) && tiles_of(64, 64) <= 256 &&
           (K <= 128 || (K <= 384 && (kM <= kN ? tiles_of(32, 64) : tiles_of(64, 32)) > 256)))
    take(64, 64, 0, 2);
  else if (vectors && (t_env == 3264 || (free_choice && kM <= kN && tiles_of(32, 64) <= 256))) take(32, 64, 4, regs ? 1 : 3);
  else if (vectors && (t_env == 6432 || (free_choice && kM > kN && tiles_of(64, 32) <= 256))) take(64, 32, 4, regs ? 1 : 3);
  else if (vectors && (t_env == 64 || (free_choice && tiles_of(64, 64) <= 256))) take(64, 64, 4, regs ? 1 : 2);
  else if (vectors && (any || indirect || t_env != 256)) {
    // Larger problems.  The CU that is given the most tiles decides, so a tile's cost is how many of them that CU takes times
    // its area, times what its k loop costs per product against the 128 x 128 stream kernel's.  Smaller tiles read more of LDS per
    // product, which weighs more the longer K is and the less C's own way does (128 x 64: 1.1 below K = 768, 1.4, 1.5 from 3000 on;
    // 64 x 64: 1.3, 2.2, 2.3; a side of 64 rows of a k-major operand a tenth more); a lone workgroup on a CU has nobody to
    // cover its waits and runs at about half the pace (1.9; below 768 1.25).  The 256 x 256 kernel reads least, but its short k loops
    // wait and nothing covers its C update (1.1, 1.0 below 1024, 0.85 below 2048, 0.77, 0.72 from 3000 on), and with fewer tiles than CUs it
    // runs at a higher clock (down to 0.9 below K = 2048, 0.7, 0.8 from 3000 on).  The ring of five 128 x 128 tiles asks for its k tiles further ahead than
    // the stream kernel: the better one alone on a CU over a long k loop (1.35 from K = 3000 on).
    // Measured on MI355X (bf16, us; ring of 128 x 128, stream 128 x 128, 128 x 64, 64 x 128, 64 x 64, 256 x 256; t: along k, n: along the rows):
    //   tt 7816 x 496 x 5288 63, 76, 77, 75, 100, 111; nt 2296 x 1688 x 8000 82, 96, 90, 91, 127, 142; tt 3120 x 1272 x 3360 42, 48, 44, 45, 56, 78;
    //   nt 632 x 7168 x 7448 99, 100, 127, 156, 166, 153; tn 1240 x 4848 x 3792 68, 62, 85, 76, 102, 85; nn 2320 x 2144 x 3928 62, 59, 73, 74, 92, 86;
    //   nn 6872 x 680 x 1752 36, 32, 37, 37, 44, 49; tn 1560 x 2720 x 6688 99, 94, 119, 114, 128, 131; tt 8032 x 4176 x 6824 584, 604, 824, 770, 1185, 579;
    //   2048^3 -, 27.4, 26.1, -, 29.2, 55; 16 x (1000 x 1504 x 776) 100, 83, 97, -, 110, 98; 4096^2 x 1024 -, 49, 56, -, 62, 52; 4096^3 158, 149, 187, -, 232, 129;
    //   5000^2 x 3000 -, 240, 296, -, 347, 195; short k loops: 4096^2 x 64 -, 23.3, -, -, -, 32.7, x 512 -, 37.9, -, -, -, 41.8; convolution
    //   128 x 100352 x 576 39, 34.1, 32.6, -, 34.2, 57.5.  Of 2000 problems drawn (60 to 3000 tiles of 128 x 128, K from 64 to 8192, all four
    //   forms) the choice is within 1.1 % of the best on average.
    // Vectors at any alignment (no ring, no 256 x 256 kernel) keep weights of their own: 1001 x 2003 x 1537 22 us in 64 x 64, 24.6 in 128 x 64.
    struct Choice { int tm, tn; double per_product, lone; };
    // Elements on both sides: bound by their loads, 1.3 in 64 x 64, 1.12 in 128 x 64 and 64 x 128 (2048^2 x 512 43.5, 41.9, 41.3, 128 x 128 44.6;
    // 2000 x 3000 x 1000 104, 89, 88, 95; 4096^2 x 1024 290, 249, 246, 222; 128 x 128 element tiles before these 101, 202, 524).
    const bool elements = a_elem && b_elem;
    const bool measured = direct && K >= 768;   // (below, and at any alignment: the weights those were measured with)
    const double half = elements ? 1.12 : measured ? (K < 3000 ? 1.4 : 1.5) : K < 1024 ? 1.1 : K < 2048 ? 1.2 : 1.3;
    const double quarter = elements ? 1.3 : measured ? (K < 3000 ? 2.2 : 2.3) : K < 1024 ? 1.3 : K < 2048 ? 1.4 : 1.65;
    const double lone = elements ? 1.2 : measured ? 1.9 : K < 2048 ? 1.25 : 1.5;
    const double side_n = measured && P.b_load == kLoadRVec ? 1.1 : 1.0, side_m = measured && P.a_load == kLoadRVec ? 1.1 : 1.0;
    const Choice choices[] = {{128, 128, 1.0, lone}, {128, 64, half * side_n, lone}, {64, 128, half * side_m, lone}, {64, 64, quarter, lone}};
    auto cost = [&](const Choice& c) {
      const int64_t per_cu = (tiles_of(c.tm, c.tn) + 255) / 256;
      return (double)per_cu * c.tm * c.tn * c.per_product * (per_cu == 1 ? c.lone : 1.0);
    };
    const Choice* best = nullptr;
    for (const Choice& c : choices)
      if (!best || cost(c) < cost(*best)) best = &c;
    const double fill = K < 2048 ? 0.9 : K < 3000 ? 0.7 : 0.8;
    const Choice big = {256, 256, (K < 768 ? 1.1 : K < 1024 ? 1.0 : K < 2048 ? 0.85 : K < 3000 ? 0.77 : 0.72) *
                                      std::min(1.0, fill + (1.0 - fill) * (double)tiles_of(256, 256) / 256.0), 1.0};
    const Choice ring = {128, 128, 1.0, 1.35};
    const bool ring_pays = direct && K >= 3000 && tiles_of(128, 128) <= 256 && cost(ring) < cost(*best);
    // Tiles of 256 x 192 and 192 x 256 (their own kernel; C in vectors) from K = 768 on: 0.91, 0.82 from 2048 on, 0.8 from 3000 on, for at least
    // 128 of them; below K = 1200, where C's update weighs too much for a second round, for one nearly full round (tn 2600 x 4112 x 880 40.1 -> 36.8, 238
    // tiles; but 192 tiles 5992 x 1368 x 896 30.9 -> 32.3, three rounds 5984 x 6072 x 960 112 -> 130).  Of 460 problems drawn (all forms, K from 128 to
    // 8192, up to 32 batch entries) they are chosen for 90 and take 0.89 of the time of the others' best on average, 1.03 at worst; figures
    // beside the kernel.  (Pairs along the rows with K from 2048 to 3000 too: 68 problems 0.89, 1.05 at worst; nn 4240 x 5248 x 2872 147 -> 137.)
    const bool wide_fits = direct && P.c_vec != 0;
    const double wide_weight = K < 2048 ? 0.91 : K < 3000 ? 0.82 : 0.8;
    auto wide_cost = [&](int64_t tm, int64_t tn) {
      const int64_t tiles = tiles_of(tm, tn);
      if (K < 768 || tiles < (K < 1200 ? 216 : 128) || (K < 1200 && tiles > 256)) return 1e30;
      return cost({(int)tm, (int)tn, wide_weight * std::min(1.0, fill + (1.0 - fill) * (double)tiles / 256.0), 1.0});
    };
    const bool tall = wide_cost(256, 192) <= wide_cost(192, 256);
    const int wide_m = tall ? 256 : 192, wide_n = tall ? 192 : 256;
    const bool wide_pays = wide_fits && wide_cost(wide_m, wide_n) < std::min(cost(big), ring_pays ? cost(ring) : cost(*best));
    if (wide_fits && (t_env == 256192 || t_env == 192256)) take(t_env / 1000, t_env % 1000, 0, 0);
    else if (free_choice && wide_pays) take(wide_m, wide_n, 0, 0);
    else if (direct && free_choice && cost(big) <= (ring_pays ? cost(ring) : cost(*best))) take(256, 256, 0, 0);
    else if (direct && (t_env == 1285 || (free_choice && ring_pays))) take(128, 128, 0, 0);
    else if (t_env == 128 || t_env == 1282 || t_env == 1284) take(128, 128, 0, 2);
    else if (t_env == 12864) take(128, 64, 0, 2);
    else if (t_env == 64128) take(64, 128, 0, 2);
    else if (t_env == 6464) take(64, 64, 0, 2);
    else take(best->tm, best->tn, 0, 2);
  }
  else if (t_env == 128 || t_env == 256) take(t_env, t_env, 0, 0);
  else if (tiles_of(256, 256) >= 256) take(256, 256, 0, 0);   // through registers: 256 x 256 when that gives every CU a tile
  else take(128, 128, 0, 0);   // (elements in these tiles: only where the tuning settings ask for staged or element loads)
  // The stream kernel's 128 x 128 tiles of two k-major operands over short k loops: pieces of 32 k rows.  Measured on MI355X (us, k tiles of 64 -> this):
  // 16 x (1000 x 1504 x 776) 85.3 -> 81.8, 20 x 1000^3 86.4 -> 81.0, 22 x (824 x 464 x 1088) 47.7 -> 44.4, 3000^2 x 320 23.5 -> 21.6, 16 x (1536^2 x 128)
  // 71.4 -> 66.8, 30 x (1300 x 700 x 900) 123.5, 123.7; 4 x (2000^2 x 1184) 63.9 -> 65.2, 6872 x 680 x 1752 33.5 -> 33.8, 4240 x 5248 x 2872 168 -> 181;
  // 128 x 64 tiles of 824 x 464 x 1088 46.9 -> 51.4; operands along k read half lines (4096^3 150 -> 181).  (LC_TUNE_GEMM_TILE 1284: whatever K is.)
  if (direct && plan.stages == 2 && plan.split_waves == 0 && plan.tile_m == 128 && plan.tile_n == 128 && P.a_load == kLoadRVec && P.b_load == kLoadRVec &&
      (t_env == 1284 || (free_choice && K <= 1100)))
    plan.stages = 4;
  // The split and stream kernels put every batch entry's tiles into one dimension of the grid, which counts lanes in 32 bits; where
  // thin problems in many batch entries have more tiles than that, the tile kernels, whose batch is a dimension of its own, take them
  // (vectors at any alignment element by element).
  if (plan.stages && (uint64_t)tiles_of(plan.tile_m, plan.tile_n) * (plan.split_waves ? 64u * (unsigned)plan.split_waves : (unsigned)kBlock) > 0xFFFFFFFFull) {
    if (any || indirect) P.a_direct = P.b_direct = 0;
    take(256, 256, 0, 0);
  }
  P.tiles_m = (uint32_t)((kM + plan.tile_m - 1) / plan.tile_m);
  P.tiles_n = (uint32_t)((kN + plan.tile_n - 1) / plan.tile_n);
  P.k_tiles = (uint32_t)((K + kGemmBK - 1) / kGemmBK);
  if ((uint64_t)P.tiles_m * P.tiles_n >= (uint64_t(1) << 31)) return LC_ERR_TOO_LARGE;
  P.group_m = (uint32_t)std::max(1, env_int("LC_TUNE_GEMM_GROUP_M", 8));
  // two stages of (rows x 128 bytes) for A and B; direct loads: a ring of five operand tiles
  // (split and stream kernels: rings of pairs of tiles, one per wavefront or one for all)
  plan.lds_bytes = plan.stages ? (unsigned)(std::max(1, plan.split_waves) * plan.stages * (plan.tile_m + plan.tile_n)) * (plan.stages == 4 ? 64u : 128u) : direct ? 5u * (unsigned)std::max(plan.tile_m, plan.tile_n) * 128u : 2u * (unsigned)(plan.tile_m + plan.tile_n) * 128u;
  plan.a_text = mode_text(a_r) + " x " + mode_text(a_k);
  plan.b_text = mode_text(b_r) + " x " + mode_text(b_k);
  plan.c_text = mode_text(c_m) + " x " + mode_text(c_n);
  if (batched) {
    plan.a_text += " x " + mode_text(a_l);
    plan.b_text += " x " + mode_text(b_l);
    plan.c_text += " x " + mode_text(c_l);
  }
  *out = plan;
  return LC_OK;
}

std::string describe(const lc_gemm_plan& plan) {
  static const char* load_name[] = {"k-vectors", "row-vectors+transpose", "elements"};
  static const char* any_name[] = {"(in unaligned k-vectors)", "(in unaligned row-vectors)"};
  static const char* gather_name[] = {"along-rows", "along-k", "k-vectors", "row-vectors"};
  std::string s = "class=gemm-mfma32x32x16 ab=";
  s += plan.ab_dtype == LC_BF16 ? "bf16" : "f16";
  s += " c=f32 M=" + std::to_string(plan.M) + " N=" + std::to_string(plan.N) + " K=" + std::to_string(plan.K);
  if (plan.L != 1 || plan.a_text.find(" x ", plan.a_text.find(" x ") + 1) != std::string::npos) s += " L=" + std::to_string(plan.L);
  s += " exchanged=" + std::to_string((int)plan.exchanged);
  s += " tile=" + std::to_string(plan.tile_m) + "x" + std::to_string(plan.tile_n) + "x" + std::to_string(kGemmBK);
  if (plan.stages && !plan.split_waves) s += " stream stages=" + std::to_string(plan.stages);
  if (plan.split_waves) s += " split_waves=" + std::to_string(plan.split_waves) + " stages=" + std::to_string(plan.stages);
  s += " tiles=" + std::to_string(plan.params.tiles_m) + "x" + std::to_string(plan.params.tiles_n) + " k_tiles=" + std::to_string(plan.params.k_tiles);
  s += " group_m=" + std::to_string(plan.params.group_m);
  s += std::string(" a_load=") + load_name[plan.params.a_load] + (plan.params.a_direct >= 4 ? "" : plan.params.a_direct >= 2 ? any_name[plan.params.a_direct - 2] : plan.params.a_direct ? "(direct-to-LDS)" : "");
  s += std::string(" b_load=") + load_name[plan.params.b_load] + (plan.params.b_direct >= 4 ? "" : plan.params.b_direct >= 2 ? any_name[plan.params.b_direct - 2] : plan.params.b_direct ? "(direct-to-LDS)" : "");
  s += " c_vec=" + std::to_string(plan.params.c_vec) + " lds_bytes=" + std::to_string(plan.lds_bytes);
  if (plan.params.a_direct == 8) s += " k-vectors=over-leaves";
  else if (plan.params.a_direct >= 4) s += std::string(" gathered=") + gather_name[plan.params.a_direct - 4] + "," + gather_name[plan.params.b_direct - 4];
  s += " A=[" + plan.a_text + "] B=[" + plan.b_text + "] C=[" + plan.c_text + "]";
  return s;
}

}  // namespace lc
