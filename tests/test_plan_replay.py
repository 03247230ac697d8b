"""The planner's routing, proven without a GPU: every plan is walked on the host along the same
index arithmetic the kernels use (bounds-checked) and compared bit for bit with the oracle's COPY."""
import time

import numpy as np
import pytest

import paper_2603_02298_amd as lc
from paper_2603_02298_amd import workloads as W


def _np_dtype(es):
    return {1: np.uint8, 2: np.uint16, 4: np.uint32, 8: np.uint64}[es]


def _check(oracle, src_layout, dst_layout, dtype, expect_class=None, seed=0):
    es = lc.DTYPE_BYTES[dtype]
    sl, dl = oracle.Layout(src_layout), oracle.Layout(dst_layout)
    rng = np.random.default_rng(seed)
    src = rng.integers(0, 255, size=sl.cosize * es, dtype=np.uint8).view(_np_dtype(es))
    want = np.full(dl.cosize, 0xA5A5A5A5A5A5A5A5 & ((1 << (8 * es)) - 1), dtype=_np_dtype(es))
    got = want.copy()
    oracle.copy(src, sl, want, dl)
    plan = lc.Plan(src_layout, dst_layout, dtype)
    desc = plan.describe()
    if expect_class:
        assert ("class=" + expect_class) in desc, desc
    conflicts = plan.debug_replay_on_host(src, got)
    assert (got == want).all(), desc
    return desc, conflicts


def test_fast_division_is_exact():
    # the kernels' division by a constant, checked through a plan whose only job is idx2crd: a
    # generic-class copy between shapes without common refinement exercises it on every element
    import ctypes
    from paper_2603_02298_amd.binding import lib
    assert lib() is not None
    rng = np.random.default_rng(1)
    # white-box: same formula as kernel_params.hpp, on random 31-bit operands
    for d in [1, 2, 3, 5, 7, 12, 64, 125, 1000, 65535, 65536, 65537, (1 << 31) - 1] + [int(x) for x in rng.integers(1, 1 << 31, 200)]:
        l = 0
        while (1 << l) < d:
            l += 1
        mul = (((1 << l) - d) << 32) // d + 1
        assert mul < (1 << 32)
        ns = np.concatenate([rng.integers(0, 1 << 31, 2000), np.array([0, 1, d - 1, d, d + 1, (1 << 31) - 1])]).astype(np.uint64)
        q = (((ns * np.uint64(mul)) >> np.uint64(32)) + ns) >> np.uint64(l)
        assert (q == ns // np.uint64(d)).all(), d


@pytest.mark.parametrize("name,scale,cls", [
    ("c1", 1, "transpose"), ("c1", 16, "transpose"), ("c2", 4, "transpose"), ("c2", 16, "transpose"),
    ("c3", 16, "transpose"), ("c4a", 64, "direct"), ("c4b", 16, "direct"), ("c5", 256, "transpose")])
def test_workloads_at_reduced_size(oracle, name, scale, cls):
    w = W.workload(name, scale)
    desc, conflicts = _check(oracle, w.src_layout, w.dst_layout, w.dtype, cls)
    if cls == "transpose":
        assert "width_bytes=16" in desc
        assert conflicts == 0, desc          # the chosen XOR swizzle is conflict-free in the bank model


def test_full_size_plans_have_expected_shape():
    # plan creation is pure host work: the full-size workloads can be planned here
    expect = {"c1": ("transpose", 16), "c2": ("transpose", 16), "c3": ("transpose", 16), "c4a": ("direct", 4),
              "c4b": ("direct", 16), "c5": ("transpose", 16)}
    for name, (cls, width) in expect.items():
        w = W.workload(name)
        d = lc.Plan(w.src_layout, w.dst_layout, w.dtype).describe()
        assert "class=%s " % cls in d and "width_bytes=%d " % width in d, d
        assert lc.Plan(w.src_layout, w.dst_layout, w.dtype).algorithmic_bytes == w.algorithmic_bytes


def test_copy_applications_table(oracle):
    from conftest import golden_lines
    for ln in golden_lines("copy_applications.txt"):
        name, s, d = [x.strip() for x in ln.split("|")]
        for dt in ("f32", "bf16", "b8", "b64"):
            desc, _ = _check(oracle, s, d, dt)
            # "Constant": every coordinate writes the one element; the loop's last write is what stays
            assert ("overwritten_modes=1" in desc) == (name == "Constant"), desc


def _random_pair(rng):
    n = int(rng.integers(1, 5))
    ext = [int(rng.choice([1, 2, 3, 4, 5, 6, 8, 12, 16])) for _ in range(n)]

    def strides(allow_zero):
        d, run = [0] * n, 1
        for m in rng.permutation(n):
            d[m] = run
            run *= ext[m] * int(rng.choice([1, 1, 1, 2, 3]))
        if allow_zero and rng.random() < 0.2:
            d[int(rng.integers(n))] = 0
        return d

    def text(exts, ds):
        # random regrouping of neighbouring modes, and random merging of compatible neighbours
        parts, i = [], 0
        while i < len(exts):
            j = min(len(exts), i + int(rng.integers(1, 3)))
            if j - i == 1:
                parts.append((str(exts[i]), str(ds[i])))
            else:
                parts.append(("(%s)" % ",".join(map(str, exts[i:j])), "(%s)" % ",".join(map(str, ds[i:j]))))
            i = j
        if len(parts) == 1:
            return "%s:%s" % parts[0]
        return "(%s):(%s)" % (",".join(p[0] for p in parts), ",".join(p[1] for p in parts))
    return text(ext, strides(True)), text(ext, strides(False))


def _random_refined_pair(rng):
    """Source and destination shapes that differ but share a refinement: a list of small factors is
    grouped into modes differently on each side (e.g. (6,4) against (2,12)); strides are compact over
    a random order of each side's own modes, sometimes padded."""
    nf = int(rng.integers(2, 6))
    factors = [int(rng.choice([2, 2, 2, 3, 4, 5, 8])) for _ in range(nf)]

    def side():
        modes, i = [], 0
        while i < nf:
            j = min(nf, i + int(rng.integers(1, 4)))
            e = 1
            for f in factors[i:j]:
                e *= f
            modes.append(e)
            i = j
        d, run = [0] * len(modes), 1
        for m in rng.permutation(len(modes)):
            d[m] = run
            run *= modes[m] * int(rng.choice([1, 1, 1, 2]))
        if len(modes) == 1:
            return "%d:%d" % (modes[0], d[0])
        return "(%s):(%s)" % (",".join(map(str, modes)), ",".join(map(str, d)))
    return side(), side()


def test_random_pairs_with_different_shapes(oracle):
    rng = np.random.default_rng(314)
    seen = {"generic": 0, "direct": 0, "transpose": 0}
    for k in range(1200):
        s, d = _random_refined_pair(rng)
        desc, _ = _check(oracle, s, d, ["f32", "bf16", "b64", "b8"][k % 4], seed=k)
        assert "note=\"shapes have no common refinement\"" not in desc, (s, d)
        seen[desc.split()[0][6:]] += 1
    assert seen["direct"] > 100 and seen["transpose"] > 100, seen


def test_random_layout_pairs(oracle):
    rng = np.random.default_rng(42)
    seen = {"generic": 0, "direct": 0, "transpose": 0}
    for k in range(1500):
        s, d = _random_pair(rng)
        dt = ["f32", "bf16", "b8", "b64", "f16"][k % 5]
        desc, _ = _check(oracle, s, d, dt, seed=k)
        seen[desc.split()[0][6:]] += 1
    assert seen["direct"] > 100 and seen["transpose"] > 100, seen


def _inner_kept_permutation(rng, es):
    """Permutation of 3-5 modes that keeps a short innermost mode in place: the common vector is a few
    16-byte words long and the copy re-orders those words (p = q)."""
    words = int(rng.choice([1, 2, 4, 8, 16]))
    inner = words * 16 // es
    n_outer = int(rng.integers(2, 5))
    ext = [inner] + [int(rng.choice([2, 3, 4, 6, 8, 12, 16, 24, 32])) for _ in range(n_outer)]
    def compact(order):
        st, run = [0] * len(ext), 1
        for m in order:
            st[m] = run
            run *= ext[m]
        return st
    so = [0] + [int(x) + 1 for x in rng.permutation(n_outer)]
    do = [0] + [int(x) + 1 for x in rng.permutation(n_outer)]
    shape = "(" + ",".join(map(str, ext)) + ")"
    return shape + ":(" + ",".join(map(str, compact(so))) + ")", shape + ":(" + ",".join(map(str, compact(do))) + ")"


def test_word_level_tiles(oracle, monkeypatch):
    # permutations that keep a short innermost mode: tiles of 16-byte words through LDS (V = 1);
    # the planner takes that route by itself from 256 tiles on (checked in the full-size plans), here it is forced
    monkeypatch.setenv("LC_TUNE_FORCE_CLASS", "2")
    desc, _ = _check(oracle, "(64,32,32,4):(1,64,2048,65536)", "(64,32,32,4):(1,2048,64,65536)", "bf16", "transpose")
    assert "V=1 tile_elem_bytes=16" in desc, desc
    desc, _ = _check(oracle, "(32,64,16,6):(1,32,2048,32768)", "(32,64,16,6):(1,512,32,32768)", "f32", "transpose")
    assert "V=1 tile_elem_bytes=16" in desc, desc
    for per_lane in (2, 4, 8):     # the tile sizes of the full-size plans
        monkeypatch.setenv("LC_TUNE_MICRO_PER_THREAD", str(per_lane))
        desc, _ = _check(oracle, "(64,32,32,4):(1,64,2048,65536)", "(64,32,32,4):(1,2048,64,65536)", "bf16", "transpose")
        assert "V=1 tile_elem_bytes=16" in desc and ("per_lane=%d" % per_lane) in desc, desc
    monkeypatch.delenv("LC_TUNE_MICRO_PER_THREAD")
    rng = np.random.default_rng(77)
    staged = 0
    for i in range(300):
        dt = ["bf16", "f32", "b8", "b64"][i % 4]
        s, d = _inner_kept_permutation(rng, lc.DTYPE_BYTES[dt])
        desc, _ = _check(oracle, s, d, dt, seed=i)
        staged += "tile_elem_bytes=16" in desc
    assert staged > 40, staged
    monkeypatch.delenv("LC_TUNE_FORCE_CLASS")
    # by itself: an attention-head permute (B,S,H,D) -> (B,H,S,D) with 128-byte heads; longer common vectors stay direct
    desc = lc.Plan("(64,32,4096,8):(1,64,2048,8388608)", "(64,32,4096,8):(1,262144,64,8388608)", "bf16").describe()
    assert "class=transpose" in desc and "V=1 tile_elem_bytes=16" in desc and "src_run_bytes=2048" in desc, desc
    desc = lc.Plan("(128,32,4096,8):(1,128,4096,16777216)", "(128,32,4096,8):(1,524288,128,16777216)", "bf16").describe()
    assert "class=direct" in desc, desc


def test_ragged_tiles(oracle):
    # extents the tile does not divide: ceil(extent / tile) tiles along the mode, coordinates checked at the edge
    for s, d, dt, want in [
        ("(67,71):(1,67)", "(67,71):(71,1)", "f32", "V=1 tile_elem_bytes=4"),          # odd transpose, no vector at all
        ("(131,77):(1,131)", "(131,77):(77,1)", "bf16", "V=1 tile_elem_bytes=2"),
        ("(45,33):(1,45)", "(45,33):(33,1)", "b8", "V=1 tile_elem_bytes=1"),
        ("(37,41):(1,37)", "(37,41):(41,1)", "b64", "V=1 tile_elem_bytes=8"),
        ("(2006,26):(1,2006)", "(2006,26):(26,1)", "f32", "V=2"),                       # 2006 = 2 * 17 * 59: whole tiles would be slivers
        ("(328,1016):(1,328)", "(328,1016):(1016,1)", "bf16", "V=8"),                   # 1016 = 8 * 127
        ("(66,50,3):(1,66,3300)", "(66,50,3):(50,1,3300)", "f32", "V=2"),                # batched
        ("(67,71,5):(1,67,4757)", "(67,71,5):(71,1,4757)", "f32", "V=1"),                 # batched, two ragged modes
    ]:
        desc, _ = _check(oracle, s, d, dt, "transpose")
        assert want in desc and "ragged_modes=0" not in desc, desc
    # power-of-two shapes keep whole tiles and the pipelined kernel
    desc, _ = _check(oracle, "(64,128):(1,64)", "(64,128):(128,1)", "f32", "transpose")
    assert "ragged_modes=0" in desc and "V=4" in desc, desc
    rng = np.random.default_rng(99)
    ragged = 0
    for i in range(250):
        M, N = int(rng.integers(9, 200)), int(rng.integers(9, 200))
        B = int(rng.choice([1, 1, 2, 3]))
        dt = ["f32", "bf16", "b8", "b64"][i % 4]
        pad = int(rng.choice([0, 0, 1, 5]))
        s = "(%d,%d,%d):(1,%d,%d)" % (M, N, B, M + pad, (M + pad) * N)
        d = "(%d,%d,%d):(%d,1,%d)" % (M, N, B, N, M * N)
        desc, _ = _check(oracle, s, d, dt, seed=i)
        ragged += "class=transpose" in desc and "ragged_modes=0" not in desc
    assert ragged > 150, ragged


def test_shapes_without_common_refinement_use_generic_class(oracle):
    for s, d in [("(2,3):(3,1)", "(3,2):(2,1)"), ("(4,9):(9,1)", "(6,6):(1,6)"), ("(5,7,3):(21,3,1)", "(3,35):(1,3)")]:
        desc, _ = _check(oracle, s, d, "f32")
    desc, _ = _check(oracle, "(6,10):(10,1)", "(4,15):(15,1)", "f32", "generic")


def test_large_copies_are_sliced_into_launches(oracle, monkeypatch):
    # work items are indexed with 31 bits; beyond that the outermost joint mode is cut into equal slices.
    # The limit is lowered here so that the slicing logic runs on sizes the host can check.
    assert "launches=4 " in lc.Plan("%d:3" % (1 << 32), "%d:1" % (1 << 32), "bf16").describe()
    assert "launches=16 " in lc.Plan("%d:1" % (1 << 36), "%d:1" % (1 << 36), "f32").describe()
    monkeypatch.setenv("LC_TUNE_MAX_ITEMS", "1000")
    monkeypatch.setenv("LC_TUNE_FORCE_CLASS", "1")       # the third case would otherwise go through element-wise tiles
    for s, d, dt, launches in [("4096:3", "4096:1", "f32", 8), ("(64,240):(1,64)", "(64,240):(1,100)", "bf16", 4),
                               ("(30,7,11):(1,30,210)", "(30,7,11):(77,11,1)", "f32", 3), ("4099:1", "4099:1", "b8", 4099)]:
        desc, _ = _check(oracle, s, d, dt, "direct")
        assert "launches=%d " % launches in desc, desc


def test_plan_errors():
    with pytest.raises(lc.LayoutCopyError) as e:
        lc.Plan("8:1", "9:1", "f32")
    assert e.value.status_name == "SIZE_MISMATCH"
    assert "class=last-writer" in lc.Plan("(4,4):(1,4)", "(4,4):(1,3)", "f32").describe()      # overlapping rows
    assert "class=" in lc.Plan("1:0", "1:0", "f32").describe()    # a single element never aliases
    assert "class=" in lc.Plan("(2,3):(3,2)", "(2,3):(3,2)", "f32").describe()   # injective though not nested


def test_destination_modes_of_stride_zero_keep_the_last_write(oracle):
    # Sec. 2.6.1's loop runs i upwards, so of the coordinates that differ only in destination modes of stride 0 the
    # last one wins: the library copies that slice (the oracle runs the loop itself)
    cases = [("(4,2):(1,4)", "(4,2):(1,0)", "f32", 1, 4),                       # the second column stays
             ("6:1", "(3,2):(1,0)", "f32", 1, 3),                                 # shapes differ: refined first
             ("(8,3,64):(1,8,24)", "(8,3,64):(64,0,1)", "bf16", 1, 16),           # a transposing copy around the dropped mode
             ("(2,5,3,4):(60,1,5,15)", "(2,5,3,4):(0,1,0,5)", "b8", 2, 60 + 2 * 5),
             ("(16,(4,2)):(1,(16,64))", "(16,(4,2)):(1,(0,16))", "b64", 1, 3 * 16),
             ("(5,7):(7,1)", "(5,7):(0,0)", "f32", 2, 34),                         # everything into one element
             ("(64,3,64):(1,4096,64)", "(64,3,64):(64,0,1)", "f32", 1, 8192)]
    for s, d, dt, modes, offset in cases:
        desc, _ = _check(oracle, s, d, dt)
        assert "overwritten_modes=%d src_offset=%d" % (modes, offset) in desc, desc
    assert "class=transpose" in _check(oracle, "(64,3,64):(1,4096,64)", "(64,3,64):(64,0,1)", "f32")[0]


def test_aliasing_destinations_keep_the_last_write(oracle):
    # Table copy, "Scatter" with repeated offsets: Sec. 2.6.1's loop leaves the value of the largest coordinate that
    # reaches an offset.  The plan is walked with both passes running BACKWARDS: only the recorded coordinates may write.
    cases = [("(4,4):(1,4)", "(4,4):(1,3)", "f32"),                         # rows that overlap by one element
             ("(4,4,2):(1,4,16)", "(4,4,2):(1,3,0)", "f32"),                # a stride-0 mode beside overlapping rows: folded first
             ("(7,5):(1,7)", "(7,5):(2,3)", "bf16"),                         # strides 2 and 3 meet often
             ("(16,16):(16,1)", "(16,16):(1,1)", "b8"),                       # anti-diagonals collapse
             ("(6,10):(10,1)", "(4,15):(3,2)", "b64"),                        # shapes without a common refinement
             ("64:1", "(8,8):(1,4)", "f32"),
             ("(3,(2,5)):(1,(3,6))", "(3,(2,5)):(5,(7,1))", "b16")]
    for s, d, dt in cases:
        desc, _ = _check(oracle, s, d, dt, "last-writer")
        assert "workspace_bytes=%d" % (4 * oracle.Layout(d).cosize) in desc or "overwritten_modes" in desc, desc
    assert "overwritten_modes=1" in lc.Plan("(4,4,2):(1,4,16)", "(4,4,2):(1,3,0)", "f32").describe()
    rng = np.random.default_rng(77)
    for i in range(200):   # random small strides on both sides: most destinations alias, some do not
        shape = [int(x) for x in rng.integers(1, 7, 3)]
        sd = [int(x) for x in rng.integers(0, 9, 3)]
        dd = [int(x) for x in rng.integers(0, 9, 3)]
        s = "(%d,%d,%d):(%d,%d,%d)" % (*shape, *sd)
        d = "(%d,%d,%d):(%d,%d,%d)" % (*shape, *dd)
        _check(oracle, s, d, ["f32", "bf16", "b8", "b64"][i % 4], seed=i)
    # a large destination whose strides do not nest is not enumerated on the host: decided per offset on the device
    big = lc.Plan("(4096,2048):(1,4096)", "(4096,2048):(3,4097)", "f32")
    assert "class=last-writer" in big.describe() and big.workspace_bytes == 4 * (4095 * 3 + 2047 * 4097 + 1)
    assert lc.Plan("(4,4):(1,4)", "(4,4):(4,1)", "f32").workspace_bytes == 0


def _check_signed(oracle, src_layout, dst_layout, dtype, seed=0):
    """_check for layouts with negative strides: both buffers extend below offset 0."""
    es = lc.DTYPE_BYTES[dtype]
    sl, dl = oracle.Layout(src_layout), oracle.Layout(dst_layout)
    so, do = -sl.min_offset, -dl.min_offset
    rng = np.random.default_rng(seed)
    src = rng.integers(0, 255, size=(so + sl.cosize) * es, dtype=np.uint8).view(_np_dtype(es))
    want = np.full(do + dl.cosize, 0xA5A5A5A5A5A5A5A5 & ((1 << (8 * es)) - 1), dtype=_np_dtype(es))
    got = want.copy()
    oracle.copy(src, sl, want, dl, src_origin=so, dst_origin=do)
    plan = lc.Plan(src_layout, dst_layout, dtype)
    plan.debug_replay_on_host(src, got, so, do)
    assert (got == want).all(), plan.describe()
    return plan.describe()


def test_negative_strides_are_planned_by_walking_modes_backwards(oracle):
    # a joint mode of negative destination stride is walked backwards on both sides (Sec. 3.4.2: any order, the same on
    # both sides): what is left has destination strides >= 0; negative source strides stay as true reversals
    d = _check_signed(oracle, "4096:1", "4096:-1", "f32")
    assert "reflected=1" in d and "dst_offset=-4095" in d and "class=direct" in d, d
    d = _check_signed(oracle, "4096:-1", "4096:-1", "f32")                      # both reversed: a plain copy again, but of the
    assert "reflected=1" in d and "joint=[(4096,1,1)]" in d and "width_bytes=4" in d, d   # memory BELOW two aligned pointers: its start is not aligned
    d = _check_signed(oracle, "4096:-1", "4096:1", "bf16")                      # a true reversal: element by element
    assert "reflected" not in d and "width_bytes=2" in d, d
    d = _check_signed(oracle, "(64,48):(1,64)", "(64,48):(-48,1)", "f32")       # transpose with flipped rows: walking the rows
    assert "reflected=1" in d and "(64,-1,48)" in d, d                          # backwards reverses the source's contiguous mode
    d = _check_signed(oracle, "(64,48):(1,-64)", "(64,48):(48,1)", "f32")       # transpose reading the columns backwards
    assert "class=transpose" in d, d
    d = _check_signed(oracle, "(256,64,3):(1,256,-16384)", "(256,64,3):(64,1,16384)", "bf16")   # batch of transposes, batches reversed
    assert "class=transpose" in d, d
    d = _check_signed(oracle, "(256,64,3):(1,256,16384)", "(256,64,3):(64,1,-16384)", "bf16")   # the same seen from the destination
    assert "class=transpose" in d and "reflected=1" in d, d
    _check_signed(oracle, "(6,10):(10,-1)", "(4,15):(-15,1)", "f32")             # no common refinement: element-wise, signed
    _check_signed(oracle, "(4,2,3):(1,4,8)", "(4,2,3):(1,0,-4)", "f32")          # an overwritten mode and a reversed one
    _check_signed(oracle, "(4,4):(1,4)", "(4,4):(-1,3)", "b16")                  # aliasing with a negative stride: last writer
    rng = np.random.default_rng(9)
    for i in range(300):
        r = int(rng.integers(1, 4))
        ext = [int(x) for x in rng.integers(1, 9, r)]
        def strides():
            order = rng.permutation(r)
            d, run = [0] * r, 1
            for m in order:
                d[m] = run * int(rng.choice([1, -1]))
                run *= ext[m] * int(rng.choice([1, 1, 2]))
            return d
        s = "(%s):(%s)" % (",".join(map(str, ext)), ",".join(map(str, strides())))
        t = "(%s):(%s)" % (",".join(map(str, ext)), ",".join(map(str, strides())))
        _check_signed(oracle, s, t, ["f32", "bf16", "b8", "b64"][i % 4], seed=i)


def test_alignment_limits_vector_width():
    wide = lc.Plan("4096:1", "4096:1", "f32").describe()
    narrow = lc.Plan("4096:1", "4096:1", "f32", src_align=4, dst_align=256).describe()
    assert "width_bytes=16" in wide and "width_bytes=4" in narrow
    # padded rows whose pitch is not a multiple of the vector: width drops to what divides it
    assert "width_bytes=8" in lc.Plan("(64,32):(1,66)", "(64,32):(1,64)", "f32").describe()
    assert "width_bytes=4" in lc.Plan("(64,32):(1,65)", "(64,32):(1,64)", "f32").describe()


def test_gather_with_small_source_stride_moves_whole_words(oracle, monkeypatch):
    """A destination-contiguous mode read with stride S (S * element < 32 bytes): 16-byte words on both sides, the lane
    keeps every S-th element of S consecutive source words.  Buffers are exactly as long as the layouts reach: the last
    vector along the mode must not read past the last element (it loads element by element).  On request only: element by
    element is faster on MI355X."""
    monkeypatch.setenv("LC_TUNE_GATHER", "1")
    cases = [("4096:3", "4096:1", "f32", 3), ("4096:2", "4096:1", "f32", 2), ("1024:7", "1024:1", "f32", 7),
             ("4096:3", "4096:1", "bf16", 3), ("2048:5", "2048:1", "bf16", 5), ("1024:7", "1024:1", "f16", 7),
             ("512:3", "512:1", "b64", 3), ("512:2", "512:1", "b64", 2),
             ("(64,30):(3,200)", "(64,30):(1,64)", "f32", 3),                 # rows of a padded matrix, every third column
             ("(32,5,7):(6,192,1920)", "(32,5,7):(1,64,320)", "bf16", 6)]     # outer strides in whole words on both sides
    for s, d, dt, stride in cases:
        desc, _ = _check(oracle, s, d, dt, "direct")
        assert "gather_stride=%d " % stride in desc and "width_bytes=16 " in desc, desc
    desc = _check_signed(oracle, "(64,9):(3,-192)", "(64,9):(1,64)", "f32")  # rows walked backwards on the source side
    assert "gather_stride=3 " in desc, desc
    # not this path: stride too long for the element width, a ragged extent, an outer stride that splits a word, a
    # broadcast mode, pointers that are not 16-byte aligned
    for s, d, dt in [("4096:8", "4096:1", "f32"), ("1024:4", "1024:1", "b64"), ("4094:3", "4094:1", "f32"),
                     ("(64,30):(3,201)", "(64,30):(1,64)", "f32"), ("(64,4):(3,0)", "(64,4):(1,64)", "f32")]:
        desc, _ = _check(oracle, s, d, dt)
        assert "gather_stride" not in desc, desc
    assert "gather_stride" not in lc.Plan("4096:3", "4096:1", "f32", src_align=4).describe()
    # sliced into launches along the gathered mode itself
    monkeypatch.setenv("LC_TUNE_MAX_ITEMS", "100")
    desc, _ = _check(oracle, "4096:3", "4096:1", "f32", "direct")
    assert "gather_stride=3 " in desc and "launches=16 " in desc, desc
    monkeypatch.delenv("LC_TUNE_MAX_ITEMS")
    monkeypatch.delenv("LC_TUNE_GATHER")
    desc, _ = _check(oracle, "4096:3", "4096:1", "f32", "direct")
    assert "gather_stride" not in desc and "width_bytes=4 " in desc, desc


@pytest.mark.parametrize("M,N,B,dt,micro", [(129, 130, 1, "f32", 1), (301, 517, 1, "bf16", 1), (64, 64, 3, "f32", 1), (65, 333, 2, "f16", 2), (1025, 36, 5, "bf16", 1),
                                            (128, 257, 1, "f32", 4), (300, 131, 1, "bf16", 1), (67, 2048, 1, "f32", 2)])
def test_shifted_tiles(oracle, monkeypatch, M, N, B, dt, micro):
    # vectors at any alignment: the last tile along a mode the tile does not divide is moved back until it ends with the mode;
    # every access of every tile stays inside buffers that are exactly as long as the layouts reach, padded sides included
    monkeypatch.setenv("LC_TUNE_SHIFTED", "1")
    monkeypatch.setenv("LC_TUNE_MICRO_PER_THREAD", str(micro))
    for pad, flip in ((0, 0), (1, 0), (3, 1)):
        s = "(%d,%d,%d):(1,%d,%d)" % (M, N, B, M + pad, (M + pad) * N)
        d = "(%d,%d,%d):(%d,1,%d)" % (M, N, B, N + pad, M * (N + pad))
        desc, conflicts = _check(oracle, *((d, s) if flip else (s, d)), dt, "transpose", seed=M + pad)
        assert "shifted_tiles=1" in desc and "width_bytes=16" in desc and conflicts == 0, desc


def test_shifted_tiles_are_the_choice_for_large_sides_that_vectors_do_not_divide(monkeypatch):
    def desc(M, N, dt, **kw):
        return lc.Plan("(%d,%d):(1,%d)" % (M, N, M), "(%d,%d):(%d,1)" % (M, N, N), dt, **kw).describe()
    assert "shifted_tiles=1" in desc(8001, 8003, "bf16") and "shifted_tiles=1" in desc(4002, 4006, "f32") and "shifted_tiles=1" in desc(8000, 8008, "bf16")
    assert "shifted_tiles=1" in desc(1024, 1024, "f32", src_align=4) and "shifted_tiles=1" in desc(4000, 4000, "bf16")
    assert "shifted" not in desc(301, 517, "bf16") and "shifted" not in desc(4000, 4000, "f32") and "shifted" not in desc(1024, 1024, "f32")
    assert "shifted" not in desc(4001, 4003, "b8") and "shifted" not in desc(2001, 2003, "b64")
    assert "shifted" not in lc.Plan("(7,1000003):(1,7)", "(7,1000003):(1000003,1)", "bf16").describe()   # a side shorter than a vector
    monkeypatch.setenv("LC_TUNE_SHIFTED", "0")
    assert "V=1" in desc(8001, 8003, "bf16")


def _nchw(N, C, hw, dt):
    return lc.Plan("(%d,%d,%d):(%d,%d,1)" % (N, C, hw, C * hw, hw), "(%d,%d,%d):(%d,1,%d)" % (N, C, hw, C * hw, C), dt).describe()


@pytest.mark.parametrize("dt,sides,pitch", [
    ("f32", (6, 4194304), 0), ("f32", (10, 4194304), 0), ("bf16", (20, 4194304), 0), ("bf16", (36, 932032), 0), ("bf16", (136, 246720), 0), ("bf16", (160, 209664), 0),
    ("bf16", (96, 349504), 0), ("f32", (36, 932032), 0), ("f32", (12, 1000004), 0), ("bf16", (68, 151200), 0), ("f32", (316, 22184), 0),
    ("bf16", (44, 746152), 64), ("bf16", (14, 354432), 64), ("f32", (48, 1368212), 64)])
def test_narrow_sides_stay_with_tiles_that_hold_them_whole(dt, sides, pitch):
    # shifted tiles would move up to twice the elements, or cut rows in two that whole tiles move at once (each measured slower)
    a, b = sides
    wide, tall = "(%d,%d):(1,%d)" % (a, b, a + pitch), "(%d,%d):(%d,1)" % (a, b, b)
    for s, d in ((wide, tall), (tall, wide)):
        desc = lc.Plan(s, d, dt).describe()
        assert "class=transpose" in desc and "shifted" not in desc, desc


def test_shifted_tiles_are_weighed_against_the_plain_plan():
    # NCHW -> NHWC of channels and images just above a tile: by the elements moved twice beyond the plain plan's own idle lanes
    for N, C, hw, dt in ((83, 256, 784, "bf16"), (1, 256, 50176, "bf16"), (594, 36, 784, "f32"), (1069, 20, 784, "f32"), (13, 24, 50176, "bf16"),
                         (1258, 68, 196, "f32"), (167, 32, 3136, "f32"), (64, 12, 16384, "bf16")):
        assert "shifted" not in _nchw(N, C, hw, dt), (N, C, hw, dt)
    for N, C, hw, dt in ((162, 132, 784, "bf16"), (648, 132, 196, "bf16"), (648, 33, 784, "bf16"), (16, 200, 12769, "f16"), (64, 256, 196, "f16"), (162, 33, 3136, "f32"),
                         (44, 24, 5776, "bf16"), (27, 232, 144, "f16"),
                         (64, 132, 61504, "f16"), (51, 52, 20164, "f16"), (21, 156, 7744, "bf16"), (1, 148, 12996, "bf16"), (50, 224, 100, "f32"),
                         (20, 196, 576, "f32"), (34, 28, 1936, "f32")):
        assert "shifted_tiles=1" in _nchw(N, C, hw, dt), (N, C, hw, dt)
    for a, b, dt in ((65, 32256, "f32"), (17, 1973760, "bf16"), (2944, 2320, "bf16"), (16, 332016, "bf16"), (3356, 11812, "f32"),
                     (8, 4040080, "bf16")):
        assert "shifted_tiles=1" in lc.Plan("(%d,%d):(1,%d)" % (a, b, a), "(%d,%d):(%d,1)" % (a, b, b), dt).describe(), (a, b, dt)
    assert "shifted_tiles=1" in lc.Plan("(60,80226):(1,68)", "(60,80226):(80226,1)", "bf16").describe()   # small gaps: the halves of a row share lines


@pytest.mark.parametrize("piece,A,B,C,wgs", [
    (48, 32, 4096, 8, 3), (96, 256, 256, 16, 3), (16, 256, 256, 16, 4), (128, 12, 3740, 6, 4), (128, 12, 7725, 3, 4), (64, 7, 9999, 9, 4), (16, 3000, 3000, 1, 4), (128, 32, 4096, 8, 4), (64, 64, 8192, 8, 2),   # tiles, by their size and number
    (16, 7, 9999, 9, 4), (32, 32, 8192, 1, 4), (48, 32, 8192, 1, 4), (16, 32, 3000, 4, 4), (128, 16, 1024, 4, 4),             # short pieces: small tiles too
    (144, 256, 256, 16, 3), (160, 32, 4096, 8, 3), (240, 1024, 1024, 1, 3),                                                  # longer ones: many tiles only
    (48, 12, 668, 8, 0), (64, 16, 1024, 4, 0), (96, 12, 668, 8, 0), (160, 32, 3000, 4, 0), (240, 32, 8192, 1, 0), (192, 64, 8192, 8, 0)])
def test_words_go_through_tiles_where_that_pays(piece, A, B, C, wgs):
    d = piece // 2
    s, t = "(%d,%d,%d,%d):(1,%d,%d,%d)" % (d, A, B, C, d, d * A, d * A * B), "(%d,%d,%d,%d):(1,%d,%d,%d)" % (d, A, B, C, d * B, d, d * A * B)
    for x, y in ((s, t), (t, s)):
        desc = lc.Plan(x, y, "bf16").describe()
        assert ("class=transpose" in desc and "V=1 " in desc) == (wgs > 0), desc
        if wgs:
            assert "wgs_per_cu=%d " % wgs in desc and "tile_queue" not in desc, desc


def test_large_windows_of_words_keep_two_items_a_lane():
    # one item and five workgroups a CU below 128 MiB, two and three from there on (rows of 512 bytes swapped over 32)
    for rows, unroll, wgs in ((2048, 1, 5), (8191, 1, 5), (8192, 2, 3), (16384, 2, 3)):
        desc = lc.Plan("(256,%d,32):(1,8192,256)" % rows, "(256,%d,32):(1,256,%d)" % (rows, 256 * rows), "bf16").describe()
        assert "class=direct" in desc and "unroll=%d " % unroll in desc and "wgs_per_cu=%d " % wgs in desc, desc


def test_tiles_of_16_byte_elements_by_their_kind():
    for a, b in ((331, 5077), (1001, 1003), (3001, 4003)):
        desc = lc.Plan("(%d,%d):(1,%d)" % (a, b, a), "(%d,%d):(%d,1)" % (a, b, b), "b128").describe()
        assert "ragged_modes=2" in desc and "wgs_per_cu=4 " in desc, desc
    assert "wgs_per_cu=4 " in lc.Plan("(1024,1024):(1,1024)", "(1024,1024):(1024,1)", "b128").describe()   # 1024 whole tiles of 16 KiB


def test_large_permutes_of_rows_run_one_item_a_lane_unless_they_step_between_channels():
    for S, H, D, unroll in ((4562, 32, 96, 1), (5775, 32, 128, 1), (5776, 32, 128, 1), (4096, 32, 128, 2), (8192, 32, 128, 2)):
        s, d = "(%d,%d,%d,6):(1,%d,%d,%d)" % (D, H, S, D, D * H, D * H * S), "(%d,%d,%d,6):(1,%d,%d,%d)" % (D, H, S, D * S, D, D * S * H)
        desc = lc.Plan(s, d, "bf16").describe()
        assert "class=direct" in desc and "unroll=%d " % unroll in desc, desc


def test_large_windows_by_their_pitch():
    for row, pitch, out_of, into in ((256, 264, 1, 1), (256, 512, 2, 2), (8192, 8200, 1, 2), (128, 136, 1, 1)):   # bf16 elements, 2^27 of them
        n = (1 << 27) // row
        a, b = "(%d,%d):(1,%d)" % (row, n, pitch), "(%d,%d):(1,%d)" % (row, n, row)
        for s, d, unroll in ((a, b, out_of), (b, a, into)):
            assert "unroll=%d " % unroll in lc.Plan(s, d, "bf16").describe(), (row, pitch, s)


PACKED_SIZES = (1, 2, 3, 4, 5, 7, 8, 9, 63, 64, 65, 1021, 4096, 100003)


@pytest.mark.parametrize("stride", range(2, 10))
def test_packed_gathers_of_16_bit_elements(oracle, monkeypatch, stride):
    # two or four elements a lane out of one load that never reaches past the last element; from stride 8 on, and for other
    # destinations and widths, one element a lane as before
    for n in PACKED_SIZES:
        desc, _ = _check(oracle, "%d:%d" % (n, stride), "%d:1" % n, "bf16")
        assert (" packed=" in desc) == (stride <= 7 and n > 1), desc
    for s, d, dt in (("64:%d" % stride, "64:1", "f32"), ("64:%d" % stride, "64:2", "bf16"), ("(64,3):(%d,1000)" % stride, "(64,3):(1,64)", "f16")):
        assert " packed=" not in _check(oracle, s, d, dt)[0]
    _check_signed(oracle, "65:-%d" % stride, "65:-1", "bf16")
    monkeypatch.setenv("LC_TUNE_PACKED", "0")
    assert " packed=" not in _check(oracle, "65:%d" % stride, "65:1", "bf16")[0]


MOVED_CASES = [  # blocks of 8 x 8 permuted, extents with few small factors; three to five modes, both widths
    ("((8,244),(8,264)):((1,8),(1952,15616))", "((8,244),(8,264)):((8,16896),(1,64))", "bf16"),      # whole tiles of few lanes
    ("((8,148),(8,188)):((1,8),(1184,9472))", "((8,148),(8,188)):((8,12032),(1,64))", "f16"),        # ragged tiles
    ("(4,61,4,1153):(4,16,1,976)", "(4,61,4,1153):(1,18448,4,16)", "f32"), ("(8,211,16,99):(211,1,26752,1688)", "(8,211,16,99):(1,12672,8,128)", "bf16"),
    ("(8,16,16,1110):(284160,16,1,256)", "(8,16,16,1110):(256,1,16,2048)", "bf16"), ("(61,8,67,9,8):(1,61,488,294264,32696)", "(61,8,67,9,8):(38592,1,576,64,8)", "bf16")]


@pytest.mark.parametrize("case", MOVED_CASES)
def test_moved_tiles(oracle, monkeypatch, case):
    # tiles cut a mode beside the two vectors' anywhere, the last one along it moved back: whole workgroups, every element
    # written and every access inside; the plan without them copies the same
    monkeypatch.setenv("LC_TUNE_SHIFTED", "2")
    desc, conflicts = _check(oracle, *case)
    assert "shifted_tiles=1" in desc and ("micro_tiles=256 " in desc), desc
    monkeypatch.delenv("LC_TUNE_SHIFTED")
    _check(oracle, *case)
    monkeypatch.setenv("LC_TUNE_MOVED", "0")
    _check(oracle, *case)


def test_where_moved_tiles_are_taken(monkeypatch):
    def desc(a, b, dt="bf16"):
        return lc.Plan("((8,%d),(8,%d)):((1,8),(%d,%d))" % (a, b, 8 * a, 64 * a), "((8,%d),(8,%d)):((8,%d),(1,64))" % (a, b, 64 * b), dt).describe()
    assert "tile=[8,8,8,32]" in desc(664, 244) and "tile=[8,8,8,32]" in desc(148, 748) and "tile=[8,8,8,32]" in desc(452, 208)
    assert "shifted_tiles" not in desc(132, 344) and "shifted_tiles" not in desc(940, 636) and "shifted_tiles" not in desc(512, 1024)
    assert "shifted_tiles" not in lc.Plan("(28,4,38576):(1,28,112)", "(28,4,38576):(154304,38576,1)", "f32").describe()   # a shorter run
    # whole tiles of 57 to 96 lanes: up to three moved tiles a CU, or in place of runs of a line and a part; 56 lanes in one round of four a CU stay
    for a, b, taken in ((480, 260, True), (312, 636, False), (464, 508, False), (600, 724, False), (476, 124, True), (392, 132, False), (644, 88, False)):
        assert ("tile=[8,8,8,32]" in desc(a, b)) == taken, (a, b)
    def moved(src, dst, dt="f32"):
        monkeypatch.delenv("LC_TUNE_MOVED", raising=False)
        taken = lc.Plan(src, dst, dt).describe()
        monkeypatch.setenv("LC_TUNE_MOVED", "0")
        return taken != lc.Plan(src, dst, dt).describe()
    # ragged fp32 tiles of the same extents: below six a CU and from twelve on
    assert moved("(40,32,4156):(4156,166240,1)", "(40,32,4156):(32,1,1280)") and moved("(4,8,1091,571):(1,4,32,34912)", "(4,8,1091,571):(4983688,1,4568,8)")
    assert not moved("(4,346,550,8):(1,4,1384,761200)", "(4,346,550,8):(2768,8,11072,1)")
    # fp32 shifted tiles with runs of 64 bytes on the destination's side stay, on the source's they go
    assert not moved("(8,74,1948):(144152,1948,1)", "(8,74,1948):(1,8,592)") and moved("(8,74,1948):(1,8,592)", "(8,74,1948):(144152,1948,1)")


def test_plans_that_moved_tiles_cannot_change_are_not_made_twice(monkeypatch):
    # where the plan in hand, or the moved tiles' extents, say no, the moved tiling is not planned to its end: making the plan takes about
    # as long with moved tiles as without (1.8 to 2.8 times as long when it was); the shortest of many, taken in turn
    for a, b in ((512, 1024), (96, 160), (640, 640)):
        src, dst = "((8,%d),(8,%d)):((1,8),(%d,%d))" % (a, b, 8 * a, 64 * a), "((8,%d),(8,%d)):((8,%d),(1,64))" % (a, b, 64 * b)
        best = {"0": 1e9, "-1": 1e9}
        for _ in range(40):
            for moved in best:
                monkeypatch.setenv("LC_TUNE_MOVED", moved)
                start = time.perf_counter()
                plan = lc.Plan(src, dst, "bf16")
                best[moved] = min(best[moved], time.perf_counter() - start)
        assert "shifted_tiles" not in plan.describe() and best["-1"] < 1.4 * best["0"], (a, b, best)


def test_workgroups_of_shifted_tiles_fill_their_rounds():
    def wgs(src, dst, dt):
        d = lc.Plan(src, dst, dt).describe()
        assert "shifted_tiles=1" in d
        return int(d.split(" tiles=")[1].split()[0]), int(d.split("wgs_per_cu=")[1].split()[0])
    def transpose(m, n, dt):
        return wgs("(%d,%d):(1,%d)" % (m, n, m), "(%d,%d):(%d,1)" % (m, n, n), dt)
    def nchw(n, c, side, dt):
        hw = side * side
        return wgs("(%d,%d,%d):(%d,%d,1)" % (n, c, hw, c * hw, hw), "(%d,%d,%d):(%d,1,%d)" % (n, c, hw, hw * c, c), dt)
    # up to five tiles a CU (256 of them): one round, or a last one that is worth its time or has so few tiles that they start beside
    # the round before it
    for tiles, w in [transpose(m, n, "bf16") for m, n in ((5967, 3033), (2821, 2883), (5169, 2367), (3321, 3451), (411, 34767), (1501, 9003))] + \
                    [transpose(m, n, "f32") for m, n in ((639, 7083), (6595, 305), (623, 4895), (1605, 1805), (2201, 1901))] + \
                    [nchw(39, 212, 44, "bf16"), nchw(48, 212, 18, "f32"), nchw(60, 84, 23, "f32")]:
        assert 256 < tiles <= 1280 and 2 <= w <= 5
        full, rest = divmod(tiles, 256 * w)
        assert full == 0 or rest <= 256 * w // 20 or rest >= 128 * w, (tiles, w)
    # runs shorter than a line: not five a CU
    assert nchw(21, 28, 174, "bf16") == (1260, 2) and nchw(13, 40, 145, "bf16") == (1092, 2)
    # far from every edge: one round of five, two of four, the last few tiles beside the round before them, long grids
    assert [transpose(m, n, "bf16") for m, n in ((5967, 3033), (4921, 6071), (2821, 2883), (5169, 2367), (6469, 7521), (4555, 8363))] == [(1128, 5), (1872, 4), (529, 2), (779, 3), (3009, 2), (2376, 2)]
    assert [transpose(m, n, "bf16") for m, n in ((7817, 2151), (5191, 3161))] == [(1054, 4), (1025, 4)] and transpose(2041, 8177, "bf16") == (1024, 4)   # one round of four, and a few more
    assert [transpose(m, n, "f32") for m, n in ((639, 7083), (1885, 4189), (8977, 5323))] == [(1110, 5), (1980, 4), (11844, 1)]
