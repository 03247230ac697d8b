"""The work this library is used for, as measurable cases: copies between layouts and GEMMs over layouts, each through the
public binding with a plan handle (or the one-shot call), on device buffers a program already holds.

A case is a dict of plain values; its `kind` names the family:
  transpose   2-D transpose, column-major to row-major, compact
  relayout    hierarchical relayout of a matrix of 8 x 8 blocks between two compact mode orders
  heads       (B,S,H,D) -> (B,H,S,D), the innermost mode kept
  nchw        NCHW -> NHWC
  gather      strided gather into a contiguous vector
  gemm        C(m,n,l) += A(m,k,l) B(n,k,l) on dense operands; `form`: t (contiguous along k) or n (along m / n) per operand
  conv        a convolution of an NHWC activation as one GEMM over its im2col view
  strided     GEMM on operands with general strides in every mode
"""
import math

import torch

import paper_2603_02298_amd as lc

_BYTES = {"f32": 4, "bf16": 2, "f16": 2}
_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def listed():
    return [
        # a small matrix transposed once between two other kernels: latency of the one-shot call and of one launch
        {"name": "transpose_small_f32", "kind": "transpose", "rows": 1024, "cols": 1024, "dtype": "f32", "call": "copy"},
        # weights repacked between two blocked storage orders, bf16
        {"name": "relayout_bf16", "kind": "relayout", "a": 512, "b": 1024, "dtype": "bf16"},
        # attention heads brought in front of the sequence, 128-byte innermost rows
        {"name": "heads_f16", "kind": "heads", "B": 8, "S": 4096, "H": 32, "D": 64, "dtype": "f16"},
        # a training batch of activations, channels last; the largest copy
        {"name": "nchw_nhwc_f32", "kind": "nchw", "N": 64, "C": 256, "H": 256, "W": 256, "dtype": "f32"},
        # a matrix whose sides nobody padded
        {"name": "transpose_odd_bf16", "kind": "transpose", "rows": 8001, "cols": 8003, "dtype": "bf16", "call": "plan"},
        # one field out of an array of three-field records
        {"name": "gather_f32", "kind": "gather", "n": 1 << 26, "stride": 3, "dtype": "f32"},
        # a small dense layer, row-major result: launch and fill of the chip
        {"name": "gemm_small_bf16", "kind": "gemm", "form": "tt", "M": 512, "N": 512, "K": 512, "L": 1, "dtype": "bf16", "c": "row"},
        # one decoding step of a dense layer: 16 rows against all of the weights
        {"name": "gemm_decode_bf16", "kind": "gemm", "form": "tt", "M": 16, "N": 8192, "K": 8192, "L": 1, "dtype": "bf16", "c": "row"},
        # a batch of ordinary matrices with ragged sides, both operands contiguous along their rows (the transposed
        # products of a backward pass)
        {"name": "gemm_batched_f16", "kind": "gemm", "form": "nn", "M": 1000, "N": 1504, "K": 776, "L": 16, "dtype": "f16", "c": "col"},
        # prefill / training size, the benchmark's
        {"name": "gemm_large_bf16", "kind": "gemm", "form": "tt", "M": 8192, "N": 8192, "K": 8192, "L": 1, "dtype": "bf16", "c": "col"},
        # a 3 x 3 convolution of 56 x 56 pixels (padded to 58), filters stored K,R,S,C
        {"name": "conv_3x3_bf16", "kind": "conv", "Nb": 32, "H": 58, "W": 58, "C": 64, "Kf": 128, "R": 3, "S": 3, "filters": "krsc", "dtype": "bf16"},
        # odd sides: no row of any operand starts on a vector boundary
        {"name": "gemm_odd_bf16", "kind": "gemm", "form": "tt", "M": 1001, "N": 2003, "K": 1537, "L": 1, "dtype": "bf16", "c": "row"},
    ]


def _log_int(rng, lo, hi, step=1):
    """An integer in [lo, hi], a multiple of step, spread over its logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def _odd(v):
    return v | 1


def draw(rng):
    kind = rng.choice(["transpose_small", "transpose_odd", "relayout", "heads", "nchw", "gather", "gemm_small", "gemm_decode", "gemm_batched",
                       "gemm_large", "conv", "gemm_odd", "strided"])
    half = rng.choice(["bf16", "f16"])
    if kind == "transpose_small":
        return {"kind": "transpose", "rows": _log_int(rng, 64, 2048, 8), "cols": _log_int(rng, 64, 2048, 8), "dtype": rng.choice(["f32", half]), "call": "copy"}
    if kind == "transpose_odd":
        return {"kind": "transpose", "rows": _odd(_log_int(rng, 257, 9000)), "cols": _odd(_log_int(rng, 257, 9000)), "dtype": rng.choice(["f32", half]), "call": "plan"}
    if kind == "relayout":
        return {"kind": "relayout", "a": _log_int(rng, 64, 1024, 4), "b": _log_int(rng, 64, 1024, 4), "dtype": half}
    if kind == "heads":
        return {"kind": "heads", "B": rng.randint(1, 8), "S": _log_int(rng, 128, 8192), "H": rng.choice([8, 12, 16, 32]), "D": rng.choice([32, 64, 80, 96, 128]), "dtype": half}
    if kind == "nchw":
        side = _log_int(rng, 7, 256)
        return {"kind": "nchw", "N": rng.randint(1, 64), "C": _log_int(rng, 8, 256, 4), "H": side, "W": side, "dtype": rng.choice(["f32", half])}
    if kind == "gather":
        return {"kind": "gather", "n": _log_int(rng, 1 << 16, 1 << 26), "stride": rng.randint(2, 8), "dtype": rng.choice(["f32", half])}
    if kind == "gemm_small":
        return {"kind": "gemm", "form": rng.choice(["tt", "nn", "nt", "tn"]), "M": _log_int(rng, 64, 1024, 8), "N": _log_int(rng, 64, 1024, 8),
                "K": _log_int(rng, 64, 1024, 8), "L": 1, "dtype": half, "c": rng.choice(["row", "col"])}
    if kind == "gemm_decode":
        return {"kind": "gemm", "form": "tt", "M": _log_int(rng, 1, 64), "N": _log_int(rng, 1024, 8192, 8), "K": _log_int(rng, 1024, 8192, 8), "L": 1,
                "dtype": half, "c": "row"}
    if kind == "gemm_batched":
        return {"kind": "gemm", "form": rng.choice(["tt", "nn"]), "M": _log_int(rng, 128, 2048, 8), "N": _log_int(rng, 128, 2048, 8), "K": _log_int(rng, 64, 2048, 8),
                "L": rng.randint(2, 32), "dtype": half, "c": rng.choice(["row", "col"])}
    if kind == "gemm_large":
        return {"kind": "gemm", "form": rng.choice(["tt", "nn", "nt"]), "M": _log_int(rng, 2048, 8192, 8), "N": _log_int(rng, 2048, 8192, 8), "K": _log_int(rng, 2048, 8192, 8),
                "L": 1, "dtype": half, "c": "col"}
    if kind == "conv":
        side = rng.randint(14, 64)
        return {"kind": "conv", "Nb": rng.randint(1, 32), "H": side, "W": side, "C": rng.choice([16, 32, 64, 128]), "Kf": _log_int(rng, 32, 256, 8), "R": 3, "S": 3,
                "filters": rng.choice(["krsc", "krsc", "kcrs"]), "dtype": half}
    if kind == "gemm_odd":
        return {"kind": "gemm", "form": rng.choice(["tt", "nn"]), "M": _odd(_log_int(rng, 101, 2049)), "N": _odd(_log_int(rng, 101, 2049)), "K": _odd(_log_int(rng, 101, 2049)),
                "L": 1, "dtype": half, "c": rng.choice(["row", "col"])}
    return {"kind": "strided", "M": _log_int(rng, 64, 1024), "N": _log_int(rng, 64, 1024), "K": _log_int(rng, 64, 1024), "dtype": half}


# ---- copies: (source layout, destination layout, source elements spanned, destination elements, source elements read) ----
def _copy_layouts(case):
    k = case["kind"]
    if k == "transpose":
        m, n = case["rows"], case["cols"]
        return "(%d,%d):(1,%d)" % (m, n, m), "(%d,%d):(%d,1)" % (m, n, n), m * n, m * n
    if k == "relayout":
        a, b = case["a"], case["b"]
        return "((8,%d),(8,%d)):((1,8),(%d,%d))" % (a, b, 8 * a, 64 * a), "((8,%d),(8,%d)):((8,%d),(1,64))" % (a, b, 64 * b), 64 * a * b, 64 * a * b
    if k == "heads":
        B, S, H, D = case["B"], case["S"], case["H"], case["D"]
        n = B * S * H * D
        return "(%d,%d,%d,%d):(1,%d,%d,%d)" % (D, H, S, B, D, D * H, D * H * S), "(%d,%d,%d,%d):(1,%d,%d,%d)" % (D, H, S, B, D * S, D, D * S * H), n, n
    if k == "nchw":
        N, C, H, W = case["N"], case["C"], case["H"], case["W"]
        n = N * C * H * W
        return ("(%d,%d,%d,%d):(%d,%d,%d,1)" % (N, C, H, W, C * H * W, H * W, W), "(%d,%d,%d,%d):(%d,1,%d,%d)" % (N, C, H, W, H * W * C, W * C, C), n, n)
    n, s = case["n"], case["stride"]
    return "%d:%d" % (n, s), "%d:1" % n, (n - 1) * s + 1, n


# ---- GEMMs: the three layouts as text, each tensor's elements, and (size, stride) lists per mode for the reference ----
def _gemm_layouts(case):
    """((text, elements, [row sizes/strides], [k or n sizes/strides], batch stride) for A, B, C), M, N, K, L."""
    if case["kind"] == "conv":
        Nb, H, W, C, Kf, R, S = (case[x] for x in ("Nb", "H", "W", "C", "Kf", "R", "S"))
        P, Q = H - R + 1, W - S + 1
        ak = [(C, R * S), (R, S), (S, 1)] if case["filters"] == "kcrs" else [(C, 1), (R, S * C), (S, C)]
        a = [(Kf, C * R * S)], ak, Kf * C * R * S, 0
        b = [(Nb, H * W * C), (P, W * C), (Q, C)], [(C, 1), (R, W * C), (S, C)], Nb * H * W * C, 0
        c = [(Kf, 1)], [(Nb, Kf * P * Q), (P, Kf * Q), (Q, Kf)], Nb * P * Q * Kf, 0
        return (a, b, c), Kf, Nb * P * Q, C * R * S, 1
    M, N, K = case["M"], case["N"], case["K"]
    if case["kind"] == "strided":   # every mode strided, none contiguous
        a = [(M, 3)], [(K, 3 * M + 1)], 3 * M + (3 * M + 1) * K, 0
        b = [(N, 2 * K + 3)], [(K, 2)], (2 * K + 3) * N + 2 * K, 0
        c = [(M, 2)], [(N, 2 * M + 1)], 2 * M + (2 * M + 1) * N, 0
        return (a, b, c), M, N, K, 1
    L, form = case["L"], case["form"]
    a = ([(M, K)], [(K, 1)], M * K * L, M * K) if form[0] == "t" else ([(M, 1)], [(K, M)], M * K * L, M * K)
    b = ([(N, K)], [(K, 1)], N * K * L, N * K) if form[1] == "t" else ([(N, 1)], [(K, N)], N * K * L, N * K)
    c = ([(M, N)], [(N, 1)], M * N * L, M * N) if case["c"] == "row" else ([(M, 1)], [(N, M)], M * N * L, M * N)
    return (a, b, c), M, N, K, L


def _mode_text(mode):
    if len(mode) == 1:
        return "%d" % mode[0][0], "%d" % mode[0][1]
    return "(" + ",".join("%d" % s for s, _ in mode) + ")", "(" + ",".join("%d" % d for _, d in mode) + ")"


def _gemm_text(tensor, L):
    r, k, _, batch = tensor
    (rs, rd), (ks, kd) = _mode_text(r), _mode_text(k)
    if L == 1:
        return "(%s,%s):(%s,%s)" % (rs, ks, rd, kd)
    return "(%s,%s,%d):(%s,%s,%d)" % (rs, ks, L, rd, kd, batch)


def _is_gemm(case):
    return case["kind"] in ("gemm", "conv", "strided")


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _gemm_inputs(case, seed):
    """N(0,1) operands and an accumulator that already holds values."""
    tensors = _gemm_layouts(case)[0]
    g = _generator(seed)
    a, b, c = (torch.randn(t[2], device="cuda", generator=g) for t in tensors)
    return a.to(_TORCH[case["dtype"]]), b.to(_TORCH[case["dtype"]]), c


def prepare(case, seed):
    stream = torch.cuda.current_stream().cuda_stream
    if _is_gemm(case):
        a, b, c = _gemm_inputs(case, seed)
        tensors, L = _gemm_layouts(case)[0], _gemm_layouts(case)[4]
        plan = lc.GemmPlan(*(_gemm_text(t, L) for t in tensors), case["dtype"])
        return {"kind": "gemm", "plan": plan, "a": a, "b": b, "c": c, "stream": stream}
    src_layout, dst_layout, src_elems, dst_elems = _copy_layouts(case)
    g = _generator(seed)
    if case["dtype"] == "f32":
        src = torch.rand(src_elems, device="cuda", generator=g).mul_(2).sub_(1)
    else:
        src = torch.randn(src_elems, device="cuda", generator=g).to(_TORCH[case["dtype"]])
    whole = torch.int32 if case["dtype"] == "f32" else torch.int16   # the copy moves bit patterns
    state = {"kind": "copy", "src": src.view(whole), "dst": torch.zeros(dst_elems, dtype=whole, device="cuda"), "stream": stream}
    if case.get("call") == "copy":
        state.update(src_layout=lc.Layout(src_layout), dst_layout=lc.Layout(dst_layout), dtype=case["dtype"])
    else:
        state["plan"] = lc.Plan(src_layout, dst_layout, case["dtype"])
    return state


def run(state):
    if state["kind"] == "gemm":
        state["plan"].execute(state["a"].data_ptr(), state["b"].data_ptr(), state["c"].data_ptr(), state["stream"])
        return state["c"]
    src, dst = state["src"].data_ptr(), state["dst"].data_ptr()
    if "plan" in state:
        state["plan"].execute(src, dst, state["stream"])
    else:
        lc.lc_copy(src, state["src_layout"], dst, state["dst_layout"], state["dtype"], state["stream"])
    return state["dst"]


def work(case):
    if _is_gemm(case):
        (a, b, c), M, N, K, L = _gemm_layouts(case)
        reads = (_conv_elems(case) if case["kind"] == "conv" else (M + N) * K * L) * 2
        return {"bytes": reads + 8 * M * N * L, "flops": 2 * M * N * K * L}   # C is read and written
    e = _BYTES[case["dtype"]]
    if case["kind"] == "gather":   # memory delivers 32-byte sectors: all of the span below 32 bytes of stride
        return {"bytes": case["n"] * (min(case["stride"] * e, 32) + e), "flops": 0}
    return {"bytes": 2 * e * _copy_layouts(case)[3], "flops": 0}


def _conv_elems(case):
    """Elements of a convolution's filters and activation."""
    return case["Kf"] * case["C"] * case["R"] * case["S"] + case["Nb"] * case["H"] * case["W"] * case["C"]


def tolerance(case):
    if not _is_gemm(case):
        return "exact"
    # exact products, sums of K terms in fp32: against 64 bits the kernels are 1e-7 to 5e-7 off (measured, K from 512 to 8192)
    return {"rel": 2e-6, "max": 2e-5}


def exact(case, seed):
    if not _is_gemm(case):
        return None
    (ta, tb, tc), M, N, K, L = _gemm_layouts(case)
    a, b, c = _gemm_inputs(case, seed)

    def matrix(t, buf, l):
        modes = t[0] + t[1]
        # the leftmost leaf of a mode runs fastest: reversed sizes make it the last axis of the view
        view = torch.as_strided(buf, [s for s, _ in reversed(t[0])] + [s for s, _ in reversed(t[1])],
                                [d for _, d in reversed(t[0])] + [d for _, d in reversed(t[1])], l * t[3])
        rows = math.prod(s for s, _ in t[0])
        return view.reshape(rows, math.prod(s for s, _ in modes) // rows)

    out = c.double()
    for l in range(L):
        product = torch.mm(matrix(ta, a, l).double().contiguous(), matrix(tb, b, l).double().t().contiguous())
        view = torch.as_strided(out, [s for s, _ in reversed(tc[0])] + [s for s, _ in reversed(tc[1])],
                                [d for _, d in reversed(tc[0])] + [d for _, d in reversed(tc[1])], l * tc[3])
        view += product.reshape(view.shape)
    return out
