"""GPU parity of the generic GEMM: the MFMA kernel (through the C ABI) against the CPU oracle on the same
seeded inputs.  Integer-valued inputs must agree exactly (every product and partial sum is exact in
fp32 whatever the order); N(0,1) inputs within K * 2^-23 * (|C0| + sum_k |A B|), the bound on fp32
accumulation of exact products in any order and rounding mode.  Run on the MI355X machine with `-m gpu`."""
import os

import numpy as np
import pytest

import paper_2603_02298_amd as lc
from paper_2603_02298_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _plan_env(env):
    class Ctx:
        def __enter__(self):
            self.old = {k: os.environ.get(k) for k in env}
            os.environ.update({k: str(v) for k, v in env.items()})

        def __exit__(self, *a):
            for k, v in self.old.items():
                if v is None:
                    del os.environ[k]
                else:
                    os.environ[k] = v
    return Ctx()


def _gpu_gemm(w, a_bits, b_bits, c0, env=None):
    dev = torch.device("cuda:0")
    tdt = torch.bfloat16 if w.ab_dtype == "bf16" else torch.float16
    a_t = torch.from_numpy(a_bits.view(np.int16)).to(dev).view(tdt)
    b_t = torch.from_numpy(b_bits.view(np.int16)).to(dev).view(tdt)
    c_t = torch.from_numpy(c0.copy()).to(dev)
    with _plan_env(env or {}):
        desc = lc.GemmPlan(w.a_layout, w.b_layout, w.c_layout, w.ab_dtype).describe()
        print("case", w.name, (w.M, w.N, w.K), desc, flush=True)
        lc.gemm_tensor(a_t, w.a_layout, b_t, w.b_layout, c_t, w.c_layout)
    torch.cuda.synchronize()
    return c_t.cpu().numpy(), desc


def _parity(oracle, w, env=None):
    a, b, c0 = W.gemm_operand_bits(w, "a"), W.gemm_operand_bits(w, "b"), W.gemm_c_values(w)
    got, desc = _gpu_gemm(w, a, b, c0, env)
    a64, b64 = W.bits_to_float64(a, w.ab_dtype), W.bits_to_float64(b, w.ab_dtype)
    want = oracle.gemm(a64, w.a_layout, b64, w.b_layout, c0.astype(np.float64), w.c_layout)
    if w.values == "ints":
        assert (got.astype(np.float64) == want).all(), desc
    else:
        bound = oracle.gemm(np.abs(a64), w.a_layout, np.abs(b64), w.b_layout, np.abs(c0).astype(np.float64), w.c_layout)
        err = np.abs(got.astype(np.float64) - want)
        assert (err <= w.K * 2.0 ** -23 * bound).all(), (desc, float(err.max()))
        # entries outside the image of C's layout keep their bits
        touched = bound != np.abs(c0).astype(np.float64)
        assert (got[~touched] == c0[~touched]).all(), desc
    return desc


# sizes the oracle finishes in seconds; each spans several tiles of the chosen size and has ragged edges
CASES = [
    ("tn", (520, 392, 200)),
    ("nt", (392, 520, 136)),
    ("nn_rowmajor_c", (264, 300, 96)),
    ("gett", (320, 200, 72)),
    ("blis", (150, 133, 77)),
]


@pytest.mark.parametrize("values", ["ints", "normal"])
@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("ktail", [0, 1])
@pytest.mark.parametrize("name,mnk", CASES)
def test_gemm_table_rows(oracle, name, mnk, tile, values, ktail):
    # K is no multiple of the k tile in any of these: ktail = 0 takes the tiles through registers (what lies past K is zeroed
    # there), ktail = 1 (the default) sends vector operands straight into LDS with zeros for the lanes past K
    w = W.gemm_workload(name, *mnk, ab_dtype="bf16", values=values)
    desc = _parity(oracle, w, {"LC_TUNE_GEMM_TILE": tile, "LC_TUNE_GEMM_KTAIL": ktail})
    assert "tile=%dx%d" % (tile, tile) in desc
    assert ("direct-to-LDS" in desc) == (ktail == 1 and name != "blis"), desc


@pytest.mark.parametrize("name,Ks", [("tn", (8, 24, 72, 200, 1000)), ("nt", (8, 40, 72, 136, 200, 1000)), ("nn_rowmajor_c", (40, 136)), ("gett", (16, 88))])
def test_gemm_short_last_k_tiles_on_the_direct_path(oracle, name, Ks):
    # the ring of LDS tiles with a last k tile that is short (from a single k on): the lanes past K present an offset out
    # of the buffer's range and zeros arrive in their slots (1285, 256: the rings of five tiles; 128: the stream kernel's two pairs)
    for K in Ks:
        for tile in (1285, 128, 256):
            for values in ("ints", "normal"):
                w = W.gemm_workload(name, 304, 264, K, ab_dtype="bf16", values=values)
                desc = _parity(oracle, w, {"LC_TUNE_GEMM_TILE": tile})
                assert desc.count("direct-to-LDS") == 2 and "k_tiles=%d " % ((K + 63) // 64) in desc, desc
                assert "tile=%dx" % (256 if tile == 256 else 128) in desc and (" stream " in desc) == (tile == 128), desc
    w = W.gemm_workload(name, 136, 200, Ks[-1], ab_dtype="f16", values="ints")
    assert "direct-to-LDS" in _parity(oracle, w)


@pytest.mark.parametrize("values", ["ints", "normal"])
def test_gemm_direct_to_lds_loads(oracle, values):
    # K a multiple of 64 and k tiles inside one leaf of the k mode: vector operands bypass the registers on their way into
    # LDS (row-vector tiles are stored k-major and read back with the LDS transpose load)
    for name, mnk in (("tn", (520, 392, 256)), ("nt", (392, 520, 192)), ("nn_rowmajor_c", (264, 300, 128)), ("gett", (320, 200, 64))):
        for tile in (128, 256):
            w = W.gemm_workload(name, *mnk, ab_dtype="bf16", values=values)
            assert "direct-to-LDS" in _parity(oracle, w, {"LC_TUNE_GEMM_TILE": tile})
    w = W.gemm_workload("tn", 200, 136, 192, ab_dtype="f16", values=values)
    assert "direct-to-LDS" in _parity(oracle, w)
    assert "direct-to-LDS" not in _parity(oracle, w, {"LC_TUNE_GEMM_DIRECT": 0})
    w = W.gemm_workload("nt", 136, 200, 128, ab_dtype="f16", values=values)
    assert "direct-to-LDS" in _parity(oracle, w)
    for name in ("tn", "nt", "nn_rowmajor_c"):   # fp16 on the 256-tile kernels
        w = W.gemm_workload(name, 392, 520, 192, ab_dtype="f16", values=values)
        desc = _parity(oracle, w, {"LC_TUNE_GEMM_TILE": 256})
        assert desc.count("direct-to-LDS") == 2 and "tile=256x256" in desc
    # k modes of several leaves whose first leaf holds whole k tiles: the tile offset steps inside the leaf and is
    # evaluated afresh at its end (A: two tiles per run, B: one)
    M, N = 200, 136
    w = W.GemmWorkload("folded_k_direct", "bf16", "(%d,(128,3)):(408,(1,136))" % M, "(%d,(64,6)):(1,(%d,%d))" % (N, N, 64 * N + 8),
                       "(%d,%d):(1,%d)" % (M, N, M), (M - 1) * 408 + 127 + 2 * 136 + 1, N + 63 * N + 5 * (64 * N + 8), M * N, M, N, 384, values)
    for tile in (128, 256):
        assert _parity(oracle, w, {"LC_TUNE_GEMM_TILE": tile}).count("direct-to-LDS") == 2
    assert "direct-to-LDS" not in _parity(oracle, w, {"LC_TUNE_GEMM_DIRECT": 1})


@pytest.mark.parametrize("K", [64, 128, 192, 256, 320])
@pytest.mark.parametrize("name", ["tn", "nt", "nn_rowmajor_c"])
def test_gemm_ring_of_tiles_with_few_k_tiles(oracle, name, K):
    # 1 to 5 k tiles through the ring of five LDS slots: the prologue requests k tiles 0, 1 and A(2) whatever K is (past
    # the last tile it repeats it), the loop's first passes run on slots the prologue filled, and with 5 tiles the
    # slots come round once.  Both sizes of the ring and the stream kernel's two pairs of tiles, integer values (exact) and N(0,1).
    for tile in (1285, 128, 256):
        for values in ("ints", "normal"):
            w = W.gemm_workload(name, 304, 264, K, ab_dtype="bf16", values=values)
            desc = _parity(oracle, w, {"LC_TUNE_GEMM_TILE": tile})
            assert desc.count("direct-to-LDS") == 2 and "k_tiles=%d " % (K // 64) in desc, desc
            assert "tile=%dx" % (256 if tile == 256 else 128) in desc and (" stream " in desc) == (tile == 128), desc


def test_gemm_f16_and_element_loads(oracle):
    for values in ("ints", "normal"):
        w = W.gemm_workload("tn", 200, 136, 104, ab_dtype="f16", values=values)
        _parity(oracle, w)
        _parity(oracle, w, {"LC_TUNE_GEMM_LOAD": 2, "LC_TUNE_GEMM_CVEC": 0})
        w = W.gemm_workload("nt", 136, 200, 64, ab_dtype="f16", values=values)
        _parity(oracle, w)


@pytest.mark.parametrize("values", ["ints", "normal"])
def test_gemm_conv_row(oracle, values):
    # the CONV row of Table gemm: a convolution as one GEMM over the im2col view of the activation
    for args in ((2, 12, 10, 3, 20, 3, 2, "kcrs"), (2, 11, 9, 8, 40, 3, 2, "krsc"), (2, 14, 12, 64, 136, 3, 3, "krsc")):
        w = W.conv_gemm_workload(*args, values=values)
        desc = _parity(oracle, w)
        assert ("direct-to-LDS" in desc) == (args[3] == 64), desc


def test_gemm_degenerate_shapes(oracle):
    # a single row / column / k, and extents below one fragment
    for M, N, K in [(1, 1, 1), (1, 40, 8), (33, 1, 5), (8, 8, 8), (31, 33, 17)]:
        w = W.gemm_workload("blis", M, N, K, values="ints")
        _parity(oracle, w)
    w = W.gemm_workload("tn", 8, 16, 8, values="ints")
    _parity(oracle, w)
    w = W.gemm_workload("nt", 8, 16, 8, values="ints")
    _parity(oracle, w)


def test_gemm_hierarchical_k_broadcast_and_accumulate(oracle):
    M, N, K1, K2 = 64, 24, 16, 3
    w = W.GemmWorkload("gett2", "bf16", "(%d,(%d,%d)):(1,(%d,%d))" % (M, K1, K2, M, M * K1 + 8),
                       "(%d,(%d,%d)):(%d,(1,%d))" % (N, K1, K2, K1, K1 * N + 16), "(%d,%d):(1,%d)" % (M, N, M),
                       (M * K1 + 8) * K2, (K1 * N + 16) * K2, M * N, M, N, K1 * K2, "ints")
    _parity(oracle, w)
    w = W.GemmWorkload("bcast", "bf16", "(40,24):(24,1)", "(16,24):(0,1)", "(40,16):(16,1)", 960, 24, 640, 40, 16, 24, "ints")
    _parity(oracle, w)
    # two executions accumulate twice (the `+=` of the loop nest)
    w = W.gemm_workload("tn", 136, 72, 40, values="ints")
    a, b, c0 = W.gemm_operand_bits(w, "a"), W.gemm_operand_bits(w, "b"), W.gemm_c_values(w)
    dev = torch.device("cuda:0")
    a_t = torch.from_numpy(a.view(np.int16)).to(dev).view(torch.bfloat16)
    b_t = torch.from_numpy(b.view(np.int16)).to(dev).view(torch.bfloat16)
    c_t = torch.from_numpy(c0.copy()).to(dev)
    lc.gemm_tensor(a_t, w.a_layout, b_t, w.b_layout, c_t, w.c_layout)
    lc.gemm_tensor(a_t, w.a_layout, b_t, w.b_layout, c_t, w.c_layout)
    torch.cuda.synchronize()
    a64, b64 = W.bits_to_float64(a, "bf16"), W.bits_to_float64(b, "bf16")
    want = oracle.gemm(a64, w.a_layout, b64, w.b_layout, c0.astype(np.float64), w.c_layout)
    want = oracle.gemm(a64, w.a_layout, b64, w.b_layout, want, w.c_layout)
    assert (c_t.cpu().numpy().astype(np.float64) == want).all()


@pytest.mark.parametrize("values", ["ints", "normal"])
@pytest.mark.parametrize("name,mnkl", [("strided_batch", (264, 136, 72, 5)), ("shared_b", (128, 300, 40, 4)),
                                       ("folded_batch", (70, 45, 33, 6)),
                                       ("strided_batch", (264, 136, 192, 3)), ("shared_b", (128, 300, 64, 4))])   # direct loads
def test_batched_gemm(oracle, name, mnkl, values):
    # the batched form of Sec. 1 (rank-3 layouts): strided batch, a shared (stride-0) operand, a folded batch mode
    w = W.batched_gemm_workload(name, *mnkl, values=values)
    desc = _parity(oracle, w)
    assert "L=%d" % w.L in desc


@pytest.mark.parametrize("name", ["tn", "nt"])
def test_gemm_full_size_sampled(oracle, name):
    # the benchmark's problem (8192^3 bf16) in the launch configuration the bench times; the oracle
    # computes sampled entries of C one by one
    M = N = K = 8192
    for values in ("ints", "normal"):
        w = W.gemm_workload(name, M, N, K, values=values)
        a, b = W.gemm_operand_bits(w, "a"), W.gemm_operand_bits(w, "b")
        c0 = W.gemm_c_values(w)
        got, desc = _gpu_gemm(w, a, b, c0)
        assert "tile=256x256" in desc
        rng = np.random.default_rng(7)
        ms = np.concatenate([rng.integers(0, M, 300), [0, M - 1, 255, 256, 4095]])
        ns = np.concatenate([rng.integers(0, N, 300), [0, N - 1, 256, 255, 4096]])
        a64, b64, c64 = W.bits_to_float64(a, "bf16"), W.bits_to_float64(b, "bf16"), c0.astype(np.float64)
        want = oracle.gemm_at(a64, w.a_layout, b64, w.b_layout, c64, w.c_layout, ms, ns)
        have = got[ms + M * ns].astype(np.float64)       # C is (M,N):(1,M)
        if values == "ints":
            assert (have == want).all(), desc
        else:
            bound = oracle.gemm_at(np.abs(a64), w.a_layout, np.abs(b64), w.b_layout, np.abs(c64), w.c_layout, ms, ns)
            assert (np.abs(have - want) <= K * 2.0 ** -23 * bound).all(), desc


@pytest.mark.parametrize("values", ["ints", "normal"])
@pytest.mark.parametrize("tile", [3216, 32, 3264, 6432, 64])
def test_gemm_split_kernel(oracle, tile, values):
    # the wavefronts of a workgroup share out the k tiles of one small tile of C: one short k tile, fewer k tiles than
    # wavefronts, more than the rings hold, ragged rows and columns, batches, both kinds of operand, C with and without vectors
    cases = [("tn", (33, 13, 8)), ("tn", (200, 16, 584)), ("tn", (1, 3, 1608)), ("nt", (40, 72, 648)), ("nn_rowmajor_c", (72, 141, 640)),
             ("gett", (192, 100, 48)), ("strided_batch", (136, 72, 104, 3)), ("shared_b", (64, 40, 24, 4))]
    for name, sizes in cases:
        w = (W.batched_gemm_workload if len(sizes) == 4 else W.gemm_workload)(name, *sizes, values=values)
        if tile == 3216 and w.N > 16:
            continue
        for env in ({}, {"LC_TUNE_GEMM_CVEC": 0}):
            assert "split_waves=" in _parity(oracle, w, dict(env, LC_TUNE_GEMM_TILE=tile))
    w = W.gemm_workload("tn", 96, 16, 200, ab_dtype="f16", values=values)
    assert "split_waves=" in _parity(oracle, w, {"LC_TUNE_GEMM_TILE": tile})


@pytest.mark.parametrize("values", ["ints", "normal"])
@pytest.mark.parametrize("tile", [128, 12864, 64128, 6464])
def test_gemm_stream_kernel(oracle, tile, values):
    # one barrier per k tile over a ring of two pairs of tiles: one to six k tiles, ragged rows and columns, batches in one
    # order with the tiles, both kinds of operand, C with and without vectors
    cases = [("tn", (200, 136, 8)), ("tn", (1, 3, 72)), ("nt", (136, 264, 328)), ("nn_rowmajor_c", (72, 141, 200)), ("gett", (192, 100, 64)),
             ("strided_batch", (136, 72, 40, 3)), ("shared_b", (128, 140, 136, 9))]
    for name, sizes in cases:
        w = (W.batched_gemm_workload if len(sizes) == 4 else W.gemm_workload)(name, *sizes, values=values)
        for env in ({}, {"LC_TUNE_GEMM_CVEC": 0}):
            assert " stream " in _parity(oracle, w, dict(env, LC_TUNE_GEMM_TILE=tile))
    w = W.conv_gemm_workload(2, 14, 12, 64, 136, 3, 3, "krsc", ab_dtype="f16", values=values)
    assert " stream " in _parity(oracle, w, {"LC_TUNE_GEMM_TILE": tile})


@pytest.mark.parametrize("values", ["ints", "normal"])
@pytest.mark.parametrize("tile", [3216, 32, 3264, 6432, 64, 128, 12864, 64128, 6464])
def test_gemm_vectors_at_any_alignment(oracle, tile, values):
    # odd sizes: 16-byte loads from any 2-byte-aligned address through registers, on the split and the stream kernel; edges
    # of vectors, tiles and k tiles, and pointers off by one element
    from test_gemm_plan import ANY_CASES, _odd_workload
    for n, case in enumerate(ANY_CASES):
        w = _odd_workload(*case, c=("col", "row")[n % 2], ab_dtype=("bf16", "f16")[n // 2 % 2], values=values)
        assert _parity(oracle, w, {"LC_TUNE_GEMM_TILE": tile}).count("elements(in unaligned") == 2
    if tile == 64:
        w = _odd_workload("tn", 72, 136, 64, values=values)
        a, b, c0 = W.gemm_operand_bits(w, "a"), W.gemm_operand_bits(w, "b"), W.gemm_c_values(w)
        dev = torch.device("cuda:0")
        a_t = torch.from_numpy(np.concatenate([a[:1], a]).view(np.int16)).to(dev).view(torch.bfloat16)[1:]
        b_t = torch.from_numpy(b.view(np.int16)).to(dev).view(torch.bfloat16)
        c_t = torch.from_numpy(c0.copy()).to(dev)
        lc.gemm_tensor(a_t, w.a_layout, b_t, w.b_layout, c_t, w.c_layout)
        a64, b64 = W.bits_to_float64(a, "bf16"), W.bits_to_float64(b, "bf16")
        want = oracle.gemm(a64, w.a_layout, b64, w.b_layout, c0.astype(np.float64), w.c_layout)
        bound = oracle.gemm(np.abs(a64), w.a_layout, np.abs(b64), w.b_layout, np.abs(c0).astype(np.float64), w.c_layout)
        assert (np.abs(c_t.cpu().numpy().astype(np.float64) - want) <= (0 if values == "ints" else w.K * 2.0 ** -23 * bound)).all()


@pytest.mark.parametrize("values", ["ints", "normal"])
@pytest.mark.parametrize("tile", [0, 32, 64, 128, 6464])
def test_gemm_vectors_at_any_alignment_in_batches_and_folded_rows(oracle, tile, values):
    from test_gemm_plan import odd_batches_and_folded_rows
    for w in odd_batches_and_folded_rows(values):
        assert _parity(oracle, w, {"LC_TUNE_GEMM_TILE": tile}).count("elements(in unaligned") == 2


@pytest.mark.parametrize("layout,rows,K", [("(2,9):(2147483638,1)", 2, 9), ("(9,9):(1,268435454)", 9, 9)])
def test_gemm_vectors_at_any_alignment_of_an_operand_that_ends_at_the_offset_limit(layout, rows, K):
    # K below a k tile and a last offset just below 2^31 (the walk of the same layouts checks every address on the host)
    L, dev = lc.Layout(layout), torch.device("cuda:0")
    far = torch.zeros(L.cosize, dtype=torch.bfloat16, device=dev)
    index = torch.tensor([[L(r + rows * k) for k in range(K)] for r in range(rows)], device=dev)
    values = torch.randint(-4, 5, (rows, K), device=dev)
    far[index] = values.to(torch.bfloat16)
    near = torch.randint(-4, 5, (3, K), device=dev)
    c = torch.zeros(rows * 3, device=dev)
    print("case", layout, flush=True)
    lc.gemm_tensor(far, layout, near.to(torch.bfloat16).ravel(), "(3,%d):(%d,1)" % (K, K), c, "(%d,3):(1,%d)" % (rows, rows))
    assert (c.reshape(3, rows).T.cpu() == (values.cpu().float() @ near.cpu().float().T)).all()


@pytest.mark.parametrize("values", ["ints", "normal"])
@pytest.mark.parametrize("tile", [0, 32, 3264, 6432, 64, 1282, 12864, 64128, 6464])
def test_gemm_gathered_operands(oracle, tile, values):
    # element by element along either mode, vectors over folded k modes, and both beside each other, on the split and stream kernels
    from test_gemm_plan import gathered_workloads
    for w, expect in gathered_workloads(values):
        assert expect in _parity(oracle, w, {"LC_TUNE_GEMM_TILE": tile})


def test_gemm_gathered_vectors_at_an_odd_pointer(oracle):
    # beside an operand of elements the vectors of the other one may start at any element
    w = W.conv_gemm_workload(1, 9, 8, 16, 40, 3, 3, "kcrs", values="ints")
    a, b, c0 = W.gemm_operand_bits(w, "a"), W.gemm_operand_bits(w, "b"), W.gemm_c_values(w)
    dev = torch.device("cuda:0")
    plan = lc.GemmPlan(w.a_layout, w.b_layout, w.c_layout, w.ab_dtype)
    assert "gathered=along-k,k-vectors" in plan.describe()
    a_t = torch.from_numpy(a.view(np.int16)).to(dev)
    c_t = torch.from_numpy(c0.copy()).to(dev)
    b_t = torch.from_numpy(np.concatenate([b[:1], b]).view(np.int16)).to(dev)[1:]
    plan.execute(a_t.data_ptr(), b_t.data_ptr(), c_t.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    want = oracle.gemm(W.bits_to_float64(a, w.ab_dtype), w.a_layout, W.bits_to_float64(b, w.ab_dtype), w.b_layout, c0.astype(np.float64), w.c_layout)
    assert (c_t.cpu().numpy().astype(np.float64) == want).all()


@pytest.mark.parametrize("values", ["ints", "normal"])
@pytest.mark.parametrize("tile", [256192, 192256])
def test_gemm_wide_tiles(oracle, tile, values):
    # the ring of 256- and 192-row tiles: one to six k tiles, short last ones, ragged edges, every pair of loads, batches, both types
    from test_gemm_plan import WIDE_CASES
    for n, (name, sizes) in enumerate(WIDE_CASES):
        w = (W.batched_gemm_workload if len(sizes) == 4 else W.gemm_workload)(name, *sizes, ab_dtype=("bf16", "f16")[n % 2], values=values)
        desc = _parity(oracle, w, {"LC_TUNE_GEMM_TILE": tile})
        assert "tile=%dx%dx64 tiles" % (tile // 1000, tile % 1000) in desc and desc.count("direct-to-LDS") == 2, desc


@pytest.mark.parametrize("values", ["ints", "normal"])
def test_gemm_pieces_of_32_k_rows(oracle, values):
    # k-major operands in k tiles of 32 through four places in LDS: every number of pieces around the ring, short last ones, both types
    for n, K in enumerate((8, 24, 32, 40, 64, 96, 104, 128, 136, 160, 328, 512)):
        w = W.gemm_workload("nt", 200, 136, K, ab_dtype=("bf16", "f16")[n % 2], values=values)
        for env in ({}, {"LC_TUNE_GEMM_CVEC": 0}):
            assert " stream stages=4" in _parity(oracle, w, dict(env, LC_TUNE_GEMM_TILE=1284))
    w = W.batched_gemm_workload("folded_batch", 33, 20, 9, 6, values=values)
    _parity(oracle, w)
