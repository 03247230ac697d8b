"""The GEMM planner and the kernel's index arithmetic, checked on the host (no GPU): plans are walked
with the library's checking device (every global access bounds-checked, tiles through a model of the
LDS arrangement and of the MFMA fragment layouts) and the result is compared with the oracle."""
import os

import numpy as np
import pytest

import paper_2603_02298_amd as lc
from paper_2603_02298_amd import workloads as W


def _walk_and_compare(oracle, w, env=None, expect=None):
    env = env or {}
    old = {k: os.environ.get(k) for k in env}
    os.environ.update({k: str(v) for k, v in env.items()})
    try:
        plan = lc.GemmPlan(w.a_layout, w.b_layout, w.c_layout, w.ab_dtype)
    finally:
        for k, v in old.items():
            if v is None:
                del os.environ[k]
            else:
                os.environ[k] = v
    text = plan.describe()
    for piece in (expect or []):
        assert piece in text, (piece, text)
    a, b, c0 = W.gemm_operand_bits(w, "a"), W.gemm_operand_bits(w, "b"), W.gemm_c_values(w)
    got = plan.debug_replay_on_host(a, b, c0.copy())
    want = oracle.gemm(W.bits_to_float64(a, w.ab_dtype), w.a_layout, W.bits_to_float64(b, w.ab_dtype), w.b_layout,
                       c0.astype(np.float64), w.c_layout)
    assert (got.astype(np.float64) == want).all(), text     # integer-valued inputs: every sum is exact
    return text


CASES = [
    # name, (M, N, K), pieces the plan's description must contain
    ("tn", (200, 136, 96), ["a_load=k-vectors", "b_load=k-vectors", "c_vec=1", "exchanged=0"]),
    ("nt", (136, 264, 72), ["a_load=row-vectors+transpose", "b_load=row-vectors+transpose", "c_vec=1"]),
    ("nn_rowmajor_c", (72, 140, 40), ["exchanged=1", "c_vec=1", "a_load=k-vectors", "b_load=row-vectors+transpose"]),
    ("gett", (192, 100, 48), ["a_load=row-vectors+transpose", "b_load=k-vectors", "c_vec=1"]),
    ("blis", (70, 45, 37), ["a_load=elements", "b_load=elements", "c_vec=0"]),
]


@pytest.mark.parametrize("name,mnk,expect", CASES)
@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("ktail", [0, 1])
def test_walk_matches_oracle(oracle, name, mnk, expect, tile, ktail):
    # K is no multiple of the k tile in any of these.  ktail = 0: tiles pass through registers, what lies past K is zeroed
    # there; ktail = 1 (the default): vector operands still go straight into LDS, the lanes past K are answered with zeros
    w = W.gemm_workload(name, *mnk, ab_dtype="bf16", values="ints")
    text = _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_TILE": tile, "LC_TUNE_GEMM_KTAIL": ktail}, expect + ["tile=%dx%d" % (tile, tile)])
    assert ("direct-to-LDS" in text) == (ktail == 1 and name != "blis"), text


def test_walk_short_last_k_tiles_on_the_direct_path(oracle):
    # K from a single vector to several tiles plus a remainder; K a multiple of 8 (no k vector may straddle K; row vectors
    # come in blocks of 8 k)
    # (1285, 256: the rings of five tiles; 128: the stream kernel)
    for name, Ks in (("tn", (8, 24, 72, 200)), ("nt", (8, 40, 72, 136, 200)), ("nn_rowmajor_c", (40, 136)), ("gett", (16, 88))):
        for K in Ks:
            for tile in (1285, 128, 256):
                w = W.gemm_workload(name, 200, 136, K, ab_dtype="bf16", values="ints")
                text = _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_TILE": tile})
                assert text.count("direct-to-LDS") == 2 and "k_tiles=%d " % ((K + 63) // 64) in text, text
                assert "tile=%dx" % (256 if tile == 256 else 128) in text and (" stream " in text) == (tile == 128), text
    w = W.gemm_workload("tn", 200, 136, 100, ab_dtype="bf16", values="ints")     # 100 = 8 * 12 + 4: a k vector would straddle K
    assert "direct" not in _walk_and_compare(oracle, w, None)


def test_walk_direct_to_lds_loads(oracle):
    # whole k tiles (K a multiple of 64, k tiles one leaf of the k mode): vector operands go straight into LDS, k-vector
    # tiles row-major, row-vector tiles k-major and read back with the LDS transpose load; the walk checks that every
    # lane's 16 bytes land in the slot the fragment reads expect, and applies the transpose load's definition
    kd, rd = "k-vectors(direct-to-LDS)", "row-vectors+transpose(direct-to-LDS)"
    for name, mnk, pieces in (("tn", (200, 136, 128), ["a_load=" + kd, "b_load=" + kd]),
                              ("nt", (136, 264, 128), ["a_load=" + rd, "b_load=" + rd]),
                              ("nn_rowmajor_c", (72, 140, 64), ["a_load=" + kd, "b_load=" + rd]),
                              ("gett", (192, 100, 64), ["a_load=" + rd, "b_load=" + kd])):
        for tile in (128, 256):
            w = W.gemm_workload(name, *mnk, ab_dtype="bf16", values="ints")
            _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_TILE": tile}, pieces)
    w = W.gemm_workload("tn", 200, 136, 128, ab_dtype="bf16", values="ints")
    assert "direct" not in _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_DIRECT": 0})
    # k modes of several leaves whose first leaf holds whole k tiles: the tile offset steps inside the leaf and is
    # evaluated afresh at its end (A: two tiles per run, B: one)
    M, N = 200, 136
    w = W.GemmWorkload("folded_k_direct", "bf16", "(%d,(128,3)):(408,(1,136))" % M, "(%d,(64,6)):(1,(%d,%d))" % (N, N, 64 * N + 8),
                       "(%d,%d):(1,%d)" % (M, N, M), (M - 1) * 408 + 127 + 2 * 136 + 1, N + 63 * N + 5 * (64 * N + 8), M * N, M, N, 384, "ints")
    _walk_and_compare(oracle, w, None, ["a_load=" + kd, "b_load=" + rd])
    # the two kinds can be switched off separately (bit 0: k vectors, bit 1: row vectors); a pair goes direct together or not at all
    w = W.gemm_workload("nt", 136, 264, 64, ab_dtype="f16", values="ints")
    assert "direct" not in _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_DIRECT": 1})
    assert "direct" in _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_DIRECT": 2})
    w = W.gemm_workload("nn_rowmajor_c", 72, 140, 64, ab_dtype="bf16", values="ints")
    assert "direct" not in _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_DIRECT": 1})


def test_walk_batched_direct_loads(oracle):
    # rank-3 layouts on the direct path: the batch offset is folded into the base the buffer loads start from
    for name, mnkl in (("strided_batch", (136, 72, 128, 3)), ("shared_b", (128, 140, 64, 2))):
        w = W.batched_gemm_workload(name, *mnkl, values="ints")
        text = _walk_and_compare(oracle, w)
        assert text.count("direct-to-LDS") == 2 and "L=%d" % w.L in text, text


def test_walk_conv_row(oracle):
    # the CONV row of Table gemm: B is the im2col view of the activation (repeated strides, not injective: fine for an
    # operand that is only read).  Filters K,C,R,S: general strides along k, element loads; filters K,R,S,C with 64
    # channels: both operands lead with whole k tiles of contiguous channels and go straight into LDS
    w = W.conv_gemm_workload(2, 6, 5, 3, 4, 3, 2, "kcrs", values="ints")
    _walk_and_compare(oracle, w, None, ["a_load=elements", "b_load=elements", "M=4 N=32 K=18"])
    w = W.conv_gemm_workload(2, 7, 6, 8, 40, 3, 2, "krsc", values="ints")
    _walk_and_compare(oracle, w, None, ["a_load=k-vectors", "b_load=k-vectors", "c_vec=1"])
    w = W.conv_gemm_workload(1, 5, 9, 64, 72, 2, 3, "krsc", values="ints")
    text = _walk_and_compare(oracle, w, None, ["a_load=k-vectors(direct-to-LDS)", "b_load=k-vectors(direct-to-LDS)"])
    assert "K=384" in text


def test_walk_f16_and_forced_element_loads(oracle):
    w = W.gemm_workload("tn", 130, 70, 40, ab_dtype="f16", values="ints")
    _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_TILE": 128}, ["ab=f16"])
    _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_TILE": 128, "LC_TUNE_GEMM_LOAD": 2, "LC_TUNE_GEMM_CVEC": 0},
                      ["a_load=elements", "b_load=elements", "c_vec=0"])


def test_walk_group_and_xcd_mapping_cover_every_tile_once(oracle):
    # 3 x 5 tiles of 128: neither a multiple of the group height nor of the 8 XCDs
    w = W.gemm_workload("tn", 300, 600, 16, ab_dtype="bf16", values="ints")
    for g in (1, 2, 4):
        _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_TILE": 128, "LC_TUNE_GEMM_GROUP_M": g}, ["tiles=3x5"])


def test_hierarchical_k_and_broadcast_operand(oracle):
    # GETT row 2 of the table: K folded as (K1,K2) with different leading leaves in A and B; and a
    # stride-0 row mode in B (every n reads the same row)
    M, N, K1, K2 = 64, 24, 16, 3
    w = W.GemmWorkload("gett2", "bf16", "(%d,(%d,%d)):(1,(%d,%d))" % (M, K1, K2, M, M * K1 + 8),
                       "(%d,(%d,%d)):(%d,(1,%d))" % (N, K1, K2, K1, K1 * N + 16), "(%d,%d):(1,%d)" % (M, N, M),
                       (M * K1 + 8) * K2, (K1 * N + 16) * K2, M * N, M, N, K1 * K2, "ints")
    _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_TILE": 128}, ["a_load=row-vectors+transpose", "b_load=k-vectors"])
    w = W.GemmWorkload("bcast", "bf16", "(40,24):(24,1)", "(16,24):(0,1)", "(40,16):(16,1)", 960, 24, 640, 40, 16, 24, "ints")
    _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_TILE": 128}, ["exchanged=1"])


@pytest.mark.parametrize("name,mnkl,expect", [
    ("strided_batch", (136, 72, 40, 3), ["L=3", "a_load=k-vectors", "b_load=k-vectors", "c_vec=1"]),
    ("shared_b", (64, 40, 24, 4), ["L=4", "a_load=row-vectors+transpose", "b_load=k-vectors", "c_vec=1"]),
    ("folded_batch", (33, 20, 9, 6), ["L=6", "a_load=elements", "exchanged=1"]),
])
def test_walk_batched_matches_oracle(oracle, name, mnkl, expect):
    # the batched form of Sec. 1: rank-3 layouts, the batch index is the second grid dimension
    w = W.batched_gemm_workload(name, *mnkl, values="ints")
    assert oracle.gemm_sizes(w.a_layout, w.b_layout, w.c_layout) == (w.M, w.N, w.K, w.L)
    _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_TILE": 128}, expect)


def test_fragment_layouts_are_the_thread_value_layouts():
    a, b, c = (lc.lc_mfma_fragment_layout(i) for i in range(3))
    assert str(a) == "((32,2),8):((1,256),32)" and str(b) == str(a) and str(c) == "((32,2),(4,4)):((32,4),(1,8))"
    # each is a bijection of (lane, value) onto the fragment's tile
    assert sorted(a(i) for i in range(512)) == list(range(512))
    assert sorted(c(i) for i in range(1024)) == list(range(1024))
    # a lane's values of A are 8 consecutive k of one row; of C, four runs of 4 consecutive rows of one column
    for lane in (0, 5, 31, 32, 63):
        ks = [a(lane + 64 * v) // 32 for v in range(8)]
        assert ks == list(range(8 * (lane // 32), 8 * (lane // 32) + 8)) and {a(lane + 64 * v) % 32 for v in range(8)} == {lane % 32}
        rows = [c(lane + 64 * v) % 32 for v in range(16)]
        assert rows == [8 * (v // 4) + 4 * (lane // 32) + v % 4 for v in range(16)]
        assert {c(lane + 64 * v) // 32 for v in range(16)} == {lane % 32}


def test_preconditions_and_refusals():
    def status(*args, **kw):
        with pytest.raises(lc.LayoutCopyError) as e:
            lc.GemmPlan(*args, **kw)
        return e.value.status_name
    assert status("(4,3):(1,4)", "(5,3):(1,5)", "(3,5):(1,3)") == "SIZE_MISMATCH"
    assert status("(4,3):(1,4)", "(5,3):(1,5)", "(4,6):(1,4)") == "SIZE_MISMATCH"
    assert status("(4,3):(1,4)", "(5,2):(1,5)", "(4,5):(1,4)") == "SIZE_MISMATCH"
    assert status("12:1", "(5,3):(1,5)", "(4,5):(1,4)") == "INVALID_ARG"
    assert status("(4,3,2):(1,4,12)", "(5,3):(1,5)", "(4,5,2):(1,4,20)") == "INVALID_ARG"            # ranks differ
    assert status("(4,3,2):(1,4,12)", "(5,3,3):(1,5,15)", "(4,5,2):(1,4,20)") == "SIZE_MISMATCH"     # batch sizes differ
    assert status("(4,3,2):(1,4,12)", "(5,3,2):(1,5,15)", "(4,5,2):(1,4,0)") == "DST_ALIASES"        # every batch entry into one C
    assert status("(4,3):(1,4)", "(5,3):(1,5)", "(4,5):(0,1)") == "DST_ALIASES"
    assert status("(4,3):(1,4)", "(5,3):(1,5)", "(4,5):(1,4)", "f32") == "UNSUPPORTED_DTYPE"
    assert status("(4,3):(1,%d)" % (1 << 30), "(5,3):(1,5)", "(4,5):(1,4)") == "TOO_LARGE"
    # less aligned pointers than vectors need: the planner falls back to element loads (for both operands
    # together) and scalar updates of C instead of refusing
    p = lc.GemmPlan("(64,64):(64,1)", "(64,64):(64,1)", "(64,64):(1,64)", "bf16", a_align=2, b_align=16, c_align=4)
    assert "a_load=elements" in p.describe() and "b_load=elements" in p.describe() and "c_vec=0" in p.describe()
    p = lc.GemmPlan("(64,64):(64,1)", "(64,64):(64,1)", "(64,64):(1,64)", "bf16", a_align=16, b_align=16, c_align=4)
    assert "a_load=k-vectors" in p.describe() and "b_load=k-vectors" in p.describe() and "c_vec=0" in p.describe()
    assert p.flops == 2 * 64 ** 3
    # execution checks the pointers against what the plan relies on before anything is launched (the addresses below
    # are never dereferenced: both calls return at the check)
    p = lc.GemmPlan("(64,64):(64,1)", "(64,64):(64,1)", "(64,64):(1,64)", "bf16")
    for ptrs in ((0x10000 + 2, 0x20000, 0x30000), (0x10000, 0x20000 + 8, 0x30000), (0x10000, 0x20000, 0x30000 + 4)):
        with pytest.raises(lc.LayoutCopyError) as e:
            p.execute(*ptrs)
        assert e.value.status_name == "MISALIGNED"
    with pytest.raises(lc.LayoutCopyError) as e:
        p.execute(0, 0x20000, 0x30000)
    assert e.value.status_name == "INVALID_ARG"


def test_lds_arrangements_are_xor_layouts_without_bank_conflicts(oracle):
    # Both LDS tile arrangements of the GEMM kernels are layouts with XOR strides (Sec. 2.3.2) over the bits of their
    # coordinates, in units of 16 bytes; and under the bank model (64 banks of 4 bytes, 256 bytes per pass) the fragment
    # reads of either arrangement touch every bank once per pass.
    from paper_2603_02298_amd.binding import lib
    addr = lib().lc_debug_gemm_lds_address
    # row-major tile: unit = 8 row + ((kv ^ row ^ (row >> 3)) & 7), coordinate (kv, row), 256 rows
    text = "((2,2,2),(2,2,2,2,2,2,2,2)):((f1,f2,f4),(f9,f18,f36,f65,f130,f260,f512,f1024))"
    for S in (oracle.SLayout, lc.SLayout):
        L = S(text)
        for row in range(256):
            for kv in range(8):
                assert 16 * L(kv + 8 * row) == addr(0, 256, 0, row, kv), (row, kv)
    # k-major tile of 256 rows (32 groups of 8 rows per k): unit = 32 k + (group ^ 4 (k mod 4)), coordinate (group, k)
    text = "((2,2,2,2,2),(2,2,2,2,2,2)):((f1,f2,f4,f8,f16),(f36,f72,f128,f256,f512,f1024))"
    for S in (oracle.SLayout, lc.SLayout):
        L = S(text)
        for k in range(64):
            for group in range(32):
                assert 16 * L(group + 32 * k) == addr(1, 256, 0, k, 8 * group), (k, group)
    # ... and of 128 rows (16 groups): the XOR reaches the top two bits of the group
    L = lc.SLayout("((2,2,2,2),(2,2,2,2,2,2)):((f1,f2,f4,f8),(f20,f40,f64,f128,f256,f512))")
    for k in range(64):
        for group in range(16):
            assert 16 * L(group + 16 * k) == addr(1, 128, 0, k, 8 * group), (k, group)

    def banks(byte_ranges):
        hit = []
        for lo, n in byte_ranges:
            assert lo % 4 == 0
            hit += [(lo // 4 + d) % 64 for d in range(n // 4)]
        return hit

    # one 16-byte read per lane, 16 lanes per pass: 16 consecutive fragment rows, one k vector
    for row0 in range(0, 256, 16):
        for kv in range(8):
            assert sorted(banks([(addr(0, 256, 0, row0 + r, kv), 16) for r in range(16)])) == list(range(64))
    # the direct loads fill 1 KiB contiguously: nothing to check.  Staged k-vector parks: lanes 0..15 = 2 rows x 8 vectors
    for row0 in range(0, 256, 2):
        assert sorted(banks([(addr(0, 256, 0, row0 + l // 8, l % 8), 16) for l in range(16)])) == list(range(64))
    # transpose loads: 8 bytes per lane, 32 lanes per pass (either half of the wavefront)
    for rows in (128, 256):
        for row_base in range(0, rows, 32):
            for k_base in range(0, 64, 4):
                for half in (0, 32):
                    got = banks([(addr(2, rows, half + l, row_base, k_base), 8) for l in range(32)])
                    assert sorted(got) == list(range(64)), (rows, row_base, k_base, half)


# (name, sizes): one short k tile; fewer k tiles than wavefronts; more than the rings hold; ragged rows, columns and batches
SPLIT_CASES = [("tn", (33, 13, 8)), ("tn", (200, 16, 584)), ("nt", (40, 72, 648)), ("nt", (8, 8, 8)), ("nn_rowmajor_c", (72, 141, 640)),
               ("gett", (192, 100, 48)), ("strided_batch", (136, 72, 40, 3)), ("shared_b", (64, 40, 24, 4))]


@pytest.mark.parametrize("tile", [3216, 32, 3264, 6432, 64])
@pytest.mark.parametrize("name,sizes", SPLIT_CASES)
def test_walk_split_kernel(oracle, name, sizes, tile):
    # workgroups whose wavefronts share out the k tiles of one small tile of C; tiles of 16 columns need at most 16
    w = (W.batched_gemm_workload if len(sizes) == 4 else W.gemm_workload)(name, *sizes, values="ints")
    if tile == 3216 and w.N > 16:
        pytest.skip("more than 16 columns")
    shape = {3216: "32x16", 3264: "32x64", 6432: "64x32"}.get(tile, "%dx%d" % (tile, tile))
    _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_TILE": tile}, [] if tile == 3216 and name != "tn" else ["tile=%sx64 split_waves=" % shape])


def test_split_kernel_is_the_choice_while_a_cu_has_at_most_one_tile_and_the_ring_for_long_k():
    def tile(M, N, K, L=1):
        d = lc.GemmPlan("(%d,%d,%d):(%d,1,%d)" % (M, K, L, K, M * K), "(%d,%d,%d):(%d,1,%d)" % (N, K, L, K, N * K), "(%d,%d,%d):(1,%d,%d)" % (M, N, L, M, M * N)).describe()
        return d.split("tile=")[1].split()[0], "split_waves" in d
    assert tile(8192, 16, 64) == ("32x16x64", True) and tile(8192, 17, 64) == ("32x32x64", True)
    assert tile(512, 512, 512) == ("32x32x64", True) and tile(516, 512, 512) == ("64x32x64", True) and tile(512, 513, 512) == ("32x64x64", True)
    assert tile(1024, 1024, 512) == ("64x64x64", True) and tile(1024, 1025, 512)[1] is False
    assert tile(1024, 1024, 64) == ("64x64x64", False) and tile(512, 513, 8) == ("64x64x64", False)   # one k tile: nothing to share
    assert tile(64, 64, 64, 64) == ("32x32x64", True) and tile(64, 64, 64, 257)[1] is False
    # with tiles for every CU either way: the stream kernel's where C's update outweighs the k loop, the ring's from K = 768 on
    assert tile(4096, 4096, 760) == ("128x128x64", False) and tile(4096, 4096, 768) == ("256x256x64", False)


def test_narrow_k_major_tiles_are_free_of_bank_conflicts():
    # k-major tiles of 32 and 64 rows: slots are a permutation of the tile, and the lanes of a transpose-load pass (32 lanes,
    # 8 bytes each) touch each of the 64 banks once
    from paper_2603_02298_amd.binding import lib
    addr = lib().lc_debug_gemm_lds_address
    for rows in (32, 64):
        assert sorted(addr(1, rows, 0, k, 8 * g) // 16 for k in range(64) for g in range(rows // 8)) == list(range(8 * rows))
        for row_base in range(0, rows, 32):
            for k_base in range(0, 64, 4):
                for half in (0, 32):
                    banks = [addr(2, rows, half + l, row_base, k_base) // 4 % 64 + d for l in range(32) for d in range(2)]
                    assert sorted(banks) == list(range(64)), (rows, row_base, k_base, half)


@pytest.mark.parametrize("tile,shape", [(128, "128x128"), (12864, "128x64"), (64128, "64x128"), (6464, "64x64")])
@pytest.mark.parametrize("name,sizes", [("tn", (200, 136, 8)), ("nt", (136, 264, 328)), ("nn_rowmajor_c", (72, 141, 200)), ("gett", (192, 100, 64)),
                                        ("strided_batch", (136, 72, 40, 3)), ("shared_b", (128, 140, 136, 9))])
def test_walk_stream_kernel(oracle, name, sizes, tile, shape):
    # one to six k tiles through a ring of two pairs of tiles, ragged rows and columns, one order over the tiles of all batch
    # entries, sums through LDS units
    w = (W.batched_gemm_workload if len(sizes) == 4 else W.gemm_workload)(name, *sizes, values="ints")
    _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_TILE": tile}, ["tile=%sx64 stream" % shape])


ANY_CASES = [  # (form, M, N, K): both along k, both along the rows, mixed; edges of vectors, tiles and k tiles; fewer rows than a vector along k
    ("tt", 33, 65, 9), ("tt", 67, 131, 129), ("tt", 5, 3, 1537), ("nn", 67, 131, 61), ("nn", 9, 11, 1), ("nn", 129, 65, 200), ("nt", 131, 70, 77),
    ("tn", 70, 131, 65), ("tt", 64, 64, 63), ("tt", 100, 72, 100), ("nt", 64, 9, 300)]


def _odd_workload(form, M, N, K, c="col", ab_dtype="bf16", values="ints"):
    a = "(%d,%d):" % (M, K) + ("(%d,1)" % K if form[0] == "t" else "(1,%d)" % M)
    b = "(%d,%d):" % (N, K) + ("(%d,1)" % K if form[1] == "t" else "(1,%d)" % N)
    return W.GemmWorkload("odd_" + form, ab_dtype, a, b, "(%d,%d):" % (M, N) + ("(1,%d)" % M if c == "col" else "(%d,1)" % N), M * K, N * K, M * N, M, N, K, values)


@pytest.mark.parametrize("tile", [0, 3216, 32, 3264, 64, 128, 64128, 6464])
@pytest.mark.parametrize("case", ANY_CASES)
def test_walk_vectors_at_any_alignment(oracle, case, tile):
    # a contiguous mode whose rows start anywhere: 16-byte loads that never leave the operand (the walk checks every one),
    # moved where they would have reached past their mode
    for c in ("col", "row"):
        text = _walk_and_compare(oracle, _odd_workload(*case, c=c), {"LC_TUNE_GEMM_TILE": tile})
        assert text.count("elements(in unaligned") == 2, text


def odd_batches_and_folded_rows(values="ints"):
    """Unaligned operands whose batch entries start at odd offsets, with one operand shared by all of them, and with a row mode of
    several leaves that hold whole vectors."""
    def w(name, dt, a, b, c, M, N, K, L=1):
        return W.GemmWorkload(name, dt, a, b, c, *(lc.Layout(x).cosize for x in (a, b, c)), M, N, K, values, "", L)
    return [
        w("odd_batch_kk", "bf16", "(33,77,3):(77,1,2543)", "(70,77,3):(77,1,5391)", "(33,70,3):(1,33,2311)", 33, 70, 77, 3),
        w("odd_batch_kr", "f16", "(67,61,4):(61,1,4089)", "(131,61,4):(1,131,7993)", "(67,131,4):(131,1,8777)", 67, 131, 61, 4),
        w("odd_batch_rr", "bf16", "(9,200,5):(1,9,1801)", "(129,200,5):(1,131,26201)", "(9,129,5):(1,9,1163)", 9, 129, 200, 5),
        w("odd_shared_b", "bf16", "(67,9,4):(9,1,605)", "(130,9,4):(9,1,0)", "(67,130,4):(1,67,8711)", 67, 130, 9, 4),
        w("odd_shared_a", "f16", "(70,75,3):(1,70,0)", "(13,75,3):(75,1,977)", "(70,13,3):(1,70,911)", 70, 13, 75, 3),
        w("folded_rows", "bf16", "((8,9),61):((1,11),99)", "(65,61):(61,1)", "(72,65):(1,72)", 72, 65, 61),
        w("folded_rows_both", "f16", "((16,5),70):((1,19),95)", "((8,17),70):((1,9),153)", "(80,136):(1,80)", 80, 136, 70)]


@pytest.mark.parametrize("tile", [0, 3216, 32, 3264, 6432, 64, 128, 12864, 64128, 6464])
def test_walk_vectors_at_any_alignment_in_batches_and_folded_rows(oracle, tile):
    for w in odd_batches_and_folded_rows():
        text = _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_TILE": tile})
        assert text.count("elements(in unaligned") == 2, text
        if tile in (128, 12864, 64128, 6464):
            assert " stream " in text, text
        elif tile in (32, 3264, 6432, 64):
            assert "split_waves" in text, text


@pytest.mark.parametrize("which,layout,expect", [("a", "(2,9):(2147483638,1)", "k-vectors"), ("a", "(2,56):(2147483591,1)", "k-vectors"),
                                                 ("a", "(9,9):(1,268435454)", "row-vectors"), ("b", "(2,9):(2147483638,1)", "k-vectors")])
def test_walk_vectors_at_any_alignment_of_an_operand_that_ends_at_the_offset_limit(which, layout, expect):
    # K below a k tile, and the operand's last offset just below 2^31: the lanes past K form no address past the operand, not
    # even on the way (the walk takes the device's 32-bit steps); the pages the walk does not touch are never made
    L = lc.Layout(layout)
    rows, K = (9, 9) if layout.startswith("(9,9)") else (2, int(layout[1:].split(")")[0].split(",")[1]))
    far = np.zeros(L.cosize, dtype=np.uint16)
    assert 2 ** 31 - 64 < far.size < 2 ** 31
    offsets = np.array([[L(r + rows * k) for k in range(K)] for r in range(rows)])
    values = np.random.default_rng(K).integers(-4, 5, (rows, K))
    far[offsets] = (values.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)   # bf16
    near = np.random.default_rng(1).integers(-4, 5, (3, K))
    near_bits = (near.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16).ravel()
    near_layout = "(3,%d):(%d,1)" % (K, K)
    c = np.zeros(rows * 3, dtype=np.float32)
    if which == "a":
        plan = lc.GemmPlan(layout, near_layout, "(%d,3):(1,%d)" % (rows, rows))
        plan.debug_replay_on_host(far, near_bits, c)
    else:
        plan = lc.GemmPlan(near_layout, layout, "(3,%d):(%d,1)" % (rows, rows))
        plan.debug_replay_on_host(near_bits, far, c)
    assert "(in unaligned %s)" % expect in plan.describe(), plan.describe()
    assert (c.reshape(3, rows).T == values @ near.T).all()


def test_which_operands_take_vectors_at_any_alignment():
    def loads(*layouts, **kw):
        d = lc.GemmPlan(*layouts, **kw).describe()
        return d.split("a_load=")[1].split(" b_load=")[0], d.split("b_load=")[1].split(" c_vec")[0]
    k, r = "elements(in unaligned k-vectors)", "elements(in unaligned row-vectors)"
    assert loads("(70,9):(9,1)", "(33,9):(1,33)", "(70,33):(33,1)") == (k, r)
    assert loads("(64,64):(64,1)", "(64,64):(1,64)", "(64,64):(1,64)", a_align=2) == (k, r)      # an aligned partner comes along
    assert loads("(70,7):(7,1)", "(33,7):(7,1)", "(70,33):(33,1)") == ("elements", "elements")   # K below one vector
    assert loads("(70,9):(9,1)", "(33,9):(3,100)", "(70,33):(33,1)") == ("elements", "elements") # a partner without a contiguous mode
    assert loads("((5,14),9):((1,5),71)", "(33,9):(9,1)", "(70,33):(33,1)") == (r, k)            # (coalesces to 70:1)
    assert loads("((5,14),9):((1,6),84)", "(33,9):(9,1)", "(70,33):(33,1)")[0] == "elements"     # vectors would straddle the leaves
    assert loads("((8,9),9):((1,9),81)", "(33,9):(9,1)", "(72,33):(33,1)")[0] == r
    assert loads("(70,(3,3)):(12,(1,4))", "(33,9):(9,1)", "(70,33):(33,1)")[0] == "elements"     # k of two leaves


def test_c_without_vectors_is_exchanged_where_the_update_passes_through_lds_only(monkeypatch):
    # C contiguous (or closer) along m, but without whole vectors of it: the split and stream kernels take that mode along n, however the
    # operands come in; the tile kernels of staged and element loads keep the roles (slower the other way round)
    def exchanged(*layouts):
        return lc.GemmPlan(*layouts).describe().split("exchanged=")[1][0]
    assert exchanged("(70,64):(64,1)", "(45,64):(64,1)", "(70,45):(1,70)") == "1" and exchanged("(70,9):(9,1)", "(45,9):(9,1)", "(70,45):(1,70)") == "1"
    assert exchanged("(70,64):(64,1)", "(16,64):(64,1)", "(70,16):(1,70)") == "0"                 # a few columns: thin tiles
    element = ("(70,9):(3,211)", "(45,9):(9,1)", "(70,45):(1,70)")
    staged = ("(35,144):(144,1)", "(450,(16,3,3)):(800,(1,32,128))", "(35,450):(1,35)")
    assert exchanged(*element) == "1" and exchanged(*staged) == "1"                               # gathered, over leaves
    assert exchanged("(1001,500):(3,3100)", "(777,500):(1100,2)", "(1001,777):(1,1001)") == "1" and exchanged("(1001,500):(3,3100)", "(777,500):(1100,2)", "(1001,777):(2,2003)") == "1"
    assert exchanged("(1001,500):(3,3100)", "(777,500):(1100,2)", "(1001,777):(1555,2)") == "0" and exchanged("(70,64):(64,1)", "(45,64):(64,1)", "(70,45):(2,141)") == "1"
    assert exchanged("(2,64):(1,2)", "(5560,64):(64,1)", "(2,5560):(1,2)") == "0" and exchanged("(56,3008):(4,224)", "(3044,3008):(9032,3)", "(56,3044):(1,57)") == "0"   # a few rows, gathered
    monkeypatch.setenv("LC_TUNE_GEMM_GATHER", "0")
    for layouts in (element, staged, ("(2,64):(1,2)", "(5560,64):(64,1)", "(2,5560):(1,2)")):
        assert exchanged(*layouts) == "0" and " stream " not in lc.GemmPlan(*layouts).describe()
    monkeypatch.delenv("LC_TUNE_GEMM_GATHER")
    assert exchanged("(70,64):(64,1)", "(45,64):(64,1)", "(70,45):(45,1)") == "0"                 # contiguous along n already


@pytest.mark.parametrize("form,M,N,K,tile", [
    # tt: both along k, nn: both along their rows (k-major tiles)
    ("nt", 632, 7168, 7448, "128x128x64 stream"), ("tn", 1240, 4848, 3792, "128x128x64 stream"), ("nn", 2320, 2144, 3928, "128x128x64 stream"),
    ("nn", 6872, 680, 1752, "128x128x64 stream"), ("nn", 4240, 5248, 2872, "256x192x64 tiles"), ("tt", 216, 34596, 1152, "128x128x64 stream"), ("tn", 5136, 776, 3008, "128x128x64 stream"), ("tn", 2248, 2240, 2704, "128x128x64 stream"),
    ("tt", 7816, 496, 5288, "128x128x64 tiles"), ("nt", 2296, 1688, 8000, "128x128x64 tiles"), ("tt", 1968, 1848, 8168, "128x128x64 tiles"),     # a lone tile on a CU, a long k loop: the ring
    ("tt", 1848, 1784, 2720, "128x64x64 stream"), ("tn", 1536, 2368, 2408, "64x128x64 stream"), ("nt", 2712, 1192, 2800, "128x64x64 stream"),    # 64 on the side that is contiguous along k
    ("tt", 4096, 4096, 4096, "256x256x64 tiles"), ("tt", 5000, 5000, 3000, "256x256x64 tiles"), ("tt", 2048, 2048, 2048, "128x64x64 stream")])
def test_tile_choice_of_middle_sizes(form, M, N, K, tile):
    # each the fastest of the tiles measured, or within 4 % of it
    a = "(%d,%d):" % (M, K) + ("(%d,1)" % K if form[0] == "t" else "(1,%d)" % M)
    b = "(%d,%d):" % (N, K) + ("(%d,1)" % K if form[1] == "t" else "(1,%d)" % N)
    text = lc.GemmPlan(a, b, "(%d,%d):(1,%d)" % (M, N, M)).describe()
    assert "tile=" + tile in text, text


@pytest.mark.parametrize("K", [8, 9])
@pytest.mark.parametrize("N,L,tile", [(53687, 40000, 0), (53684, 40000, 0), (16385, 65535, 32), (16385, 65535, 3264), (16385, 65535, 6464)])
def test_thin_problems_in_many_batch_entries_fit_a_grid(K, N, L, tile, monkeypatch):
    # one row in tens of thousands of batch entries: more than 2^24 tiles, and one dimension of a grid holds no more workgroups of 256
    # lanes; the kernels with the batch in a dimension of its own take them
    if tile:
        monkeypatch.setenv("LC_TUNE_GEMM_TILE", str(tile))
    text = lc.GemmPlan("(1,%d,%d):(%d,1,%d)" % (K, L, K, K), "(%d,%d,%d):(%d,1,0)" % (N, K, L, K), "(1,%d,%d):(1,1,%d)" % (N, L, N)).describe()
    tiles_m, tiles_n = (int(x) for x in text.split(" tiles=")[1].split()[0].split("x"))
    assert " stream " not in text and "split_waves" not in text and "tile=256x256" in text and tiles_m * tiles_n * 256 < 2 ** 32, text
    assert ("direct-to-LDS" in text) == (K == 8) and "unaligned" not in text, text


def test_as_many_tiles_as_one_dimension_of_a_grid_holds(monkeypatch):
    monkeypatch.setenv("LC_TUNE_GEMM_TILE", "6464")
    text = lc.GemmPlan("(1,8,65535):(8,1,8)", "(16384,8,65535):(8,1,0)", "(1,16384,65535):(1,1,16384)").describe()
    assert " stream " in text and "L=65535" in text and "tiles=256x1 " in text, text   # 256 x 65535 workgroups of 256 lanes


def gathered_workloads(values="ints"):
    """Operands that vectors along one mode of a single leaf do not cover, on either side or both: general strides, filters stored
    K,C,R,S beside an activation in vectors, channels too few for a k tile, odd channels, folded k modes of row vectors."""
    def w(name, dt, a, b, c, M, N, K, L=1):
        return W.GemmWorkload(name, dt, a, b, c, *(lc.Layout(x).cosize for x in (a, b, c)), M, N, K, values, "", L)
    return [
        (W.gemm_workload("blis", 70, 45, 37, values=values), "gathered=along-k,along-rows"),
        (W.gemm_workload("blis", 131, 67, 200, ab_dtype="f16", values=values), "gathered=along-k,along-rows"),
        (W.conv_gemm_workload(1, 9, 8, 16, 40, 3, 3, "kcrs", values=values), "gathered=along-k,k-vectors"),
        (W.conv_gemm_workload(2, 8, 7, 72, 33, 3, 3, "kcrs", ab_dtype="f16", values=values), "gathered=along-k,k-vectors"),
        (W.conv_gemm_workload(1, 7, 8, 5, 33, 3, 3, "krsc", values=values), "gathered=along-k,along-k"),
        (W.conv_gemm_workload(2, 9, 8, 24, 44, 3, 3, "krsc", values=values), "k-vectors=over-leaves"),
        (W.conv_gemm_workload(1, 12, 9, 8, 136, 3, 3, "krsc", ab_dtype="f16", values=values), "k-vectors=over-leaves"),
        (W.conv_gemm_workload(1, 8, 8, 96, 70, 2, 3, "krsc", values=values), "k-vectors=over-leaves"),
        # 14, 23 and 35 k tiles, the last one short: past the 12 and 16 places of the split kernel's rings, and several a wavefront through registers
        (W.conv_gemm_workload(1, 6, 7, 96, 45, 3, 3, "krsc", values=values), "k-vectors=over-leaves"),
        (W.conv_gemm_workload(1, 7, 6, 160, 72, 3, 3, "krsc", ab_dtype="f16", values=values), "k-vectors=over-leaves"),
        (W.conv_gemm_workload(1, 6, 6, 248, 36, 3, 3, "krsc", values=values), "k-vectors=over-leaves"),
        (W.conv_gemm_workload(1, 6, 6, 248, 33, 3, 3, "kcrs", values=values), "gathered=along-k,k-vectors"),
        (w("folded_k_rows", "bf16", "(72,(8,9)):(1,(80,704))", "(136,(8,9)):(1,(136,1200))", "(72,136):(1,72)", 72, 136, 72), "gathered=row-vectors,row-vectors"),
        (w("folded_k_mixed", "f16", "(72,(8,9)):(1,(80,704))", "(33,(8,9)):(3,(100,1100))", "(72,33):(1,72)", 72, 33, 72), "gathered=row-vectors,along-rows"),
        (w("folded_k_kr", "bf16", "(65,(16,5)):(104,(1,20))", "(40,(16,5)):(5,(203,4000))", "(65,40):(41,1)", 65, 40, 80), "gathered=along-k,along-rows"),
        (w("batched", "bf16", "(33,20,3):(61,3,2101)", "(40,20,3):(1,41,0)", "(33,40,3):(1,35,1501)", 33, 40, 20, 3), "gathered=along-k,along-rows"),
        (w("reversed_lead", "f16", "(1,9):(9,2)", "(7,9):(2,15)", "(1,7):(1,3)", 1, 7, 9), "gathered=")]


@pytest.mark.parametrize("tile", [0, 32, 3264, 6432, 64, 1282, 12864, 64128, 6464])
def test_walk_gathered_operands(oracle, tile):
    # eight elements (or a vector) a lane, every address inside the operand, in the slot the fragments are read from
    for w, expect in gathered_workloads():
        _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_TILE": tile}, [expect, "split_waves=" if tile in (32, 3264, 6432, 64) else "tile="])


def test_choice_of_short_k_loops_and_of_vectors_over_folded_k():
    def text(M, N, K):
        return lc.GemmPlan("(%d,%d):(%d,1)" % (M, K, K), "(%d,%d):(%d,1)" % (N, K, K), "(%d,%d):(1,%d)" % (M, N, M)).describe()
    # several k tiles, but too few to share out: the stream kernel's 64 x 64 tiles
    for M, N, K, stream in ((800, 800, 72, True), (800, 800, 384, True), (800, 800, 392, False), (800, 400, 128, True), (800, 400, 136, False), (512, 512, 72, False)):
        assert (" stream " in text(M, N, K)) == stream, (M, N, K)
    def folded(M, K):   # row vectors on both sides, k of two leaves
        return lc.GemmPlan(*["(%d,(32,%d)):(1,(%d,%d))" % (M, K // 32, M, 33 * M)] * 2, "(%d,%d):(1,%d)" % (M, M, M)).describe()
    assert "gathered=row-vectors,row-vectors" in folded(1920, 320) and "gathered" not in folded(2048, 320)
    def leaves(M, K):   # k vectors on both sides, k of two leaves
        return lc.GemmPlan(*["(%d,(32,%d)):(%d,(1,40))" % (M, K // 32, 40 * K // 32)] * 2, "(%d,%d):(1,%d)" % (M, M, M)).describe()
    assert "over-leaves" in leaves(4096, 2976) and "over-leaves" in leaves(3840, 3008) and "over-leaves" not in leaves(4096, 3008)


WIDE_CASES = [("tn", (300, 200, 8)), ("nt", (264, 400, 136)), ("nn_rowmajor_c", (200, 300, 200)), ("gett", (320, 200, 64)), ("tn", (388, 396, 320)),
              ("nt", (200, 264, 384)), ("strided_batch", (136, 72, 40, 3)), ("shared_b", (256, 192, 200, 2))]


@pytest.mark.parametrize("tile,shape", [(256192, "256x192"), (192256, "192x256")])
def test_walk_wide_tiles(oracle, tile, shape):
    # one to six k tiles through a ring whose slots hold tiles of 256 and of 192 rows, short last k tiles, ragged rows and columns
    for name, sizes in WIDE_CASES:
        w = (W.batched_gemm_workload if len(sizes) == 4 else W.gemm_workload)(name, *sizes, values="ints")
        _walk_and_compare(oracle, w, {"LC_TUNE_GEMM_TILE": tile}, ["tile=%sx64 tiles" % shape, "lds_bytes=163840"])


def test_k_major_tiles_of_192_rows_are_free_of_bank_conflicts():
    from paper_2603_02298_amd.binding import lib
    addr = lib().lc_debug_gemm_lds_address
    assert sorted(addr(1, 192, 0, k, 8 * g) // 16 for k in range(64) for g in range(24)) == list(range(8 * 192))
    for row_base in range(0, 192, 32):
        for k_base in range(0, 64, 4):
            for half in (0, 32):
                banks = [addr(2, 192, half + l, row_base, k_base) // 4 % 64 + d for l in range(32) for d in range(2)]
                assert sorted(banks) == list(range(64)), (row_base, k_base, half)


def test_where_wide_tiles_are_taken():
    def tile(form, M, N, K, c="col", L=1):
        a = "(%d,%d):" % (M, K) + ("(%d,1)" % K if form[0] == "t" else "(1,%d)" % M)
        b = "(%d,%d):" % (N, K) + ("(%d,1)" % K if form[1] == "t" else "(1,%d)" % N)
        return lc.GemmPlan(a, b, "(%d,%d):" % (M, N) + ("(1,%d)" % M if c == "col" else "(%d,1)" % N)).describe().split("tile=")[1].split("x64 ")[0]
    assert tile("nt", 3368, 5336, 6576) == "256x192" and tile("tt", 1872, 5312, 2008) == "192x256" and tile("tn", 2600, 4112, 880) == "192x256" and tile("tt", 5656, 2968, 8048) == "256x192"
    assert tile("tt", 1872, 5312, 760) == "128x64" and tile("nt", 5984, 6072, 960) == "128x128" and tile("tt", 1816, 5256, 5080) == "192x256" and tile("tt", 8192, 8192, 8192) == "256x256" and tile("nn", 4376, 4376, 4808) == "256x192"
    assert tile("tt", 3370, 5336, 6576) not in ("256x192", "192x256")   # C without vectors


def test_walk_pieces_of_32_k_rows(oracle):
    # one to eleven pieces through four places in LDS, short last ones, ragged rows and columns, batches
    for name, sizes in [("nt", (200, 136, K)) for K in (8, 24, 32, 40, 64, 72, 96, 104, 136, 328)] + [("nt", (128, 264, 200))]:
        _walk_and_compare(oracle, W.gemm_workload(name, *sizes, values="ints"), {"LC_TUNE_GEMM_TILE": 1284}, ["tile=128x128x64 stream stages=4", "lds_bytes=65536"])
    def stages(form, M, N, K, L):
        a = "(%d,%d,%d):" % (M, K, L) + ("(%d,1,%d)" % (K, M * K) if form[0] == "t" else "(1,%d,%d)" % (M, M * K))
        b = "(%d,%d,%d):" % (N, K, L) + ("(%d,1,%d)" % (K, N * K) if form[1] == "t" else "(1,%d,%d)" % (N, N * K))
        return lc.GemmPlan(a, b, "(%d,%d,%d):(1,%d,%d)" % (M, N, L, M, M * N)).describe()
    assert [" stream stages=4 " in stages(f, 1000, 1504, K, 16) for f, K in (("nn", 776), ("nn", 1096), ("nn", 1104), ("tt", 776), ("tn", 776))] == [True, True, False, False, False]
