"""Performance cases of the CCL GEMM framework: the calls a training or
serving program makes, through the public entry points of
paper_2606_11718_amd.ccl.

A case is one of three kinds:

  gemm  one GEMM C = alpha A B + beta C of an FFN layer. The activations (A,
        and B too in a weight gradient, "b_live") arrive row-major or as the
        stored transpose and are packed in the pass; weights are packed
        beforehand. C is handed back row-major ("unpack") or stays in CCL.
  ffn   the whole forward FFN, Y = (X W_up) W_down, with the intermediate
        kept in CCL.
  pack  a weight or activation matrix brought into CCL: row-major, from the
        stored transpose, or both, and optionally back.

Sizes are the repository's own workloads (an expert FFN of 2048 hidden and
2 x 768 intermediate, a dense FFN of 8192 hidden and 28672 intermediate) and
generic ones around them.
"""
from __future__ import annotations

import torch

from paper_2606_11718_amd import ccl

DEV = "cuda"
AB = {"bf16": (ccl.CCL_DT_BF16, torch.bfloat16, 2), "fp8": (ccl.CCL_DT_FP8_E4M3, torch.float8_e4m3fn, 1),
      "fp32": (ccl.CCL_DT_FP32, torch.float32, 4)}
CT = {"bf16": (ccl.CCL_DT_BF16, torch.bfloat16, 2), "fp32": (ccl.CCL_DT_FP32, torch.float32, 4)}

# Standard deviations of the operands: activations N(0,1), weights N(0,0.02),
# gradients N(0,0.01). fp8 weights are stored scaled up to N(0,1), and the
# GEMM's alpha scales the product back.
ACT, WEIGHT, GRAD = 1.0, 0.02, 0.01


def _gemm(name, M, N, K, **more):
    case = {"name": name, "kind": "gemm", "M": M, "N": N, "K": K, "chiplets": 8, "grid": 0, "page": 4096,
            "ab": "bf16", "c": "bf16", "a_trans": False, "b_live": False, "splitk": False, "alpha": 1.0,
            "beta": 0.0, "unpack": True, "ld_pad": 0, "a_std": ACT, "b_std": WEIGHT}
    case.update(more)
    return case


def _ffn(name, M, D, F, **more):
    case = {"name": name, "kind": "ffn", "M": M, "D": D, "F": F, "chiplets": 8, "grid": 2, "page": 4096,
            "splitk": False}
    case.update(more)
    return case


def _pack(name, M, N, K, **more):
    case = {"name": name, "kind": "pack", "M": M, "N": N, "K": K, "op": "B", "chiplets": 8, "grid": 2,
            "page": 4096, "ab": "bf16", "rows": True, "trans": True, "unpack": False, "ld_pad": 0}
    case.update(more)
    return case


def listed():
    return [
        # The smallest configuration of the repository: three dependent
        # launches of a few microseconds each.
        _gemm("tiny_forward", 256, 512, 256, chiplets=4, grid=2, a_std=0.58, b_std=0.58),
        # Expert FFN, fused gate and up projection, 4096 tokens, forward.
        _gemm("expert_gate_up", 4096, 1536, 2048, grid=2),
        # Expert FFN backward: the down projection's weight gradient H^T dY
        # (H as stored, long K, few output tiles: split-K) ...
        _gemm("expert_dw_down", 768, 2048, 4096, a_trans=True, b_live=True, splitk=True, b_std=GRAD),
        # ... and the gradient of its input, dY W_down^T.
        _gemm("expert_dh", 4096, 768, 2048, a_std=GRAD),
        # The same expert forward with fp8 operands and a dequantising scale.
        _gemm("expert_gate_up_fp8", 4096, 1536, 2048, grid=2, ab="fp8", alpha=0.02, b_std=1.0),
        # Weight gradient from a ragged number of tokens (13 * 256) with an
        # odd number of output tiles.
        _gemm("ragged_dw", 1152, 2048, 3328, a_trans=True, b_live=True, b_std=GRAD),
        # Ragged prefill: 15 * 128 tokens, read out of a wider activation
        # buffer.
        _gemm("ragged_forward", 1920, 5120, 1792, ld_pad=8),
        # Dense FFN, one decode batch of 128 tokens: bound by reading the
        # weights.
        _ffn("dense_ffn_decode", 128, 8192, 28672, grid=1, splitk=True),
        # Dense FFN prefill of 8192 tokens: the headline step.
        _ffn("dense_ffn_prefill", 8192, 8192, 28672),
        # Dense FFN up projection with fp8 operands; the result stays in CCL
        # for the next layer.
        _gemm("dense_up_fp8", 8192, 28672, 8192, grid=2, ab="fp8", alpha=0.02, b_std=1.0, unpack=False),
        # Dense FFN backward: the up projection's weight gradient X^T dY,
        # accumulated over micro-batches into an fp32 buffer kept in CCL.
        _gemm("dense_dw_up_accumulate", 8192, 28672, 8192, grid=1, c="fp32", beta=1.0, a_trans=True,
              b_live=True, b_std=GRAD, unpack=False),
        # A dense weight after an optimizer step, packed for the forward pass
        # and, transposed, for the backward pass.
        _pack("dense_weight_pack", 1024, 28672, 8192),
    ]


def _log(rng, lo, hi):
    """A whole number of lo..hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def _shape(rng, grid, max_flops):
    """M, N, K on a grid x 8/grid partition with whole 128 x 128 tiles and K
    blocks of whole 64-element steps or, for odd multiples of 256, halves."""
    cols = 8 // grid
    while True:
        M = 128 * grid * _log(rng, 1, 128 // grid)
        N = 128 * cols * _log(rng, 1, 224 // cols)
        K = 256 * _log(rng, 2, 112)
        if 2.0 * M * N * K <= max_flops:
            return M, N, K


def draw(rng):
    """One more case of the same ranges: 128 to 16384 tokens, 128 to 28672
    columns, K from 512 to 28672, every grid, page size and direction."""
    kind = rng.choice(["forward", "forward", "forward_fp8", "dx", "dw", "dw", "dw_accumulate", "ffn", "decode", "pack"])
    grid = rng.choice([1, 2, 4, 8])
    page = rng.choice([4096, 4096, 65536, 2 * 1024 * 1024])
    pad = rng.choice([0, 0, 0, 8, 8, 2 * rng.randint(0, 40) + 1])
    M, N, K = _shape(rng, grid, 1.5e12)
    if kind == "forward":
        case = _gemm("", M, N, K, grid=grid, page=page, ld_pad=pad, unpack=rng.random() < 0.6)
    elif kind == "forward_fp8":
        K = 512 * max(1, K // 512)
        case = _gemm("", M, N, K, grid=grid, page=page, ab="fp8", alpha=0.02, b_std=1.0, ld_pad=pad, unpack=rng.random() < 0.6)
    elif kind == "dx":
        case = _gemm("", M, N, K, grid=grid, page=page, ld_pad=pad, a_std=GRAD)
    elif kind == "dw":
        case = _gemm("", M, N, K, grid=grid, page=page, ld_pad=pad, a_trans=True, b_live=True, b_std=GRAD, splitk=rng.random() < 0.7)
    elif kind == "dw_accumulate":
        case = _gemm("", M, N, K, grid=grid, page=page, ld_pad=pad, a_trans=True, b_live=True, b_std=GRAD, c="fp32", beta=1.0, unpack=False)
    elif kind == "ffn":
        cols = 8 // grid
        D, F = 256 * cols * _log(rng, 1, 32 // cols), 256 * cols * _log(rng, 1, 112 // cols)
        case = _ffn("", M, D, F, grid=grid, page=page)
    elif kind == "decode":
        D, F = 2048 * rng.randint(1, 4), 2048 * rng.randint(1, 14)
        case = _ffn("", 128 * _log(rng, 1, 4), D, F, grid=1, page=page, splitk=True)
    else:
        op = rng.choice(["A", "B"])
        if op == "A":
            K = 8 * rng.randint(64, 3584)
        else:
            K = 1024 * _log(rng, 1, 28)
        ab = rng.choice(["bf16", "bf16", "fp8", "fp32"])
        rows = rng.random() < 0.7
        case = _pack("", M, N, K, op=op, grid=grid, page=page, ab=ab, rows=rows, trans=not rows or rng.random() < 0.5,
                     unpack=rng.random() < 0.5, ld_pad=pad)
    del case["name"]
    return case


# ---- inputs, plans and buffers ---------------------------------------------

def _normal(seed, index, rows, cols, std, ab):
    """A rows x cols matrix of N(0, std) values in the type ab."""
    g = torch.Generator(device=DEV).manual_seed(1000 * seed + index)
    dtype = AB[ab][1]
    x = torch.randn(rows, cols, generator=g, device=DEV, dtype=torch.float32 if ab == "fp32" else torch.bfloat16).mul_(std)
    return x.to(dtype)


def _wide(x, pad):
    """x as the leading columns of a buffer with pad more columns."""
    if not pad:
        return x
    out = torch.empty(x.shape[0], x.shape[1] + pad, device=x.device, dtype=x.dtype)
    out[:, :x.shape[1]] = x
    return out[:, :x.shape[1]]


def _plan(case, M, N, K, ab="bf16", c="bf16"):
    return ccl.ccl_plan_typed(M, N, K, case["chiplets"], case["grid"], case["page"], AB[ab][0], CT[c][0])


def _buffer(plan, op, dtype):
    lay = ccl.ccl_plan_layout(plan, op)
    return torch.zeros(lay.total_bytes, dtype=torch.uint8, device=DEV).view(dtype)


def _source(case, seed, index, rows, cols, std, trans=False, pad=0):
    """The stored matrix of a rows x cols operand: itself, or its transpose."""
    shape = (cols, rows) if trans else (rows, cols)
    return _wide(_normal(seed, index, *shape, std, case.get("ab", "bf16")), pad)


def _split_state(plan, wanted):
    """Split-K ranges and workspace a program sets up with its plan."""
    if not wanted:
        return 1, None, 0
    ranges, need = ccl.ccl_gemm_splitk_workspace(plan, 0)
    return ranges, (torch.empty(need, dtype=torch.uint8, device=DEV) if need else None), need


def prepare(case, seed):
    return {"gemm": _prepare_gemm, "ffn": _prepare_ffn, "pack": _prepare_pack}[case["kind"]](case, seed)


def _prepare_gemm(case, seed):
    M, N, K, ab, c = case["M"], case["N"], case["K"], case["ab"], case["c"]
    plan = _plan(case, M, N, K, ab, c)
    st = {"case": case, "plan": plan}
    st["a_src"] = _source(case, seed, 1, M, K, case["a_std"], case["a_trans"], case["ld_pad"])
    st["a"] = _buffer(plan, ccl.CCL_A, AB[ab][1])
    b = _source(case, seed, 2, K, N, case["b_std"])
    st["b"] = _buffer(plan, ccl.CCL_B, AB[ab][1])
    if case["b_live"]:
        st["b_src"] = b
    else:
        ccl.ccl_pack(plan, ccl.CCL_B, b, N, 0, st["b"])
    st["c"] = _buffer(plan, ccl.CCL_C, CT[c][1])
    if case["beta"]:
        c0 = _normal(seed, 3, M, N, 1.0, c)
        ccl.ccl_pack(plan, ccl.CCL_C, c0, N, 0, st["c"])
    if case["unpack"]:
        st["out"] = torch.empty(M, N, dtype=CT[c][1], device=DEV)
    st["ranges"], st["ws"], st["ws_bytes"] = _split_state(plan, case["splitk"])
    return st


def _prepare_ffn(case, seed):
    M, D, F = case["M"], case["D"], case["F"]
    up, down = _plan(case, M, F, D), _plan(case, M, D, F)
    st = {"case": case, "up": up, "down": down, "x_src": _normal(seed, 1, M, D, ACT, "bf16")}
    st["w_up"], st["w_down"] = (_buffer(p, ccl.CCL_B, torch.bfloat16) for p in (up, down))
    ccl.ccl_pack(up, ccl.CCL_B, _normal(seed, 2, D, F, WEIGHT, "bf16"), F, 0, st["w_up"])
    ccl.ccl_pack(down, ccl.CCL_B, _normal(seed, 3, F, D, WEIGHT, "bf16"), D, 0, st["w_down"])
    st["x"], st["h"] = (_buffer(up, op, torch.bfloat16) for op in (ccl.CCL_A, ccl.CCL_C))
    st["y"] = _buffer(down, ccl.CCL_C, torch.bfloat16)
    st["out"] = torch.empty(M, D, dtype=torch.bfloat16, device=DEV)
    st["up_split"], st["down_split"] = (_split_state(p, case["splitk"]) for p in (up, down))
    return st


def _pack_plans(case):
    """The plan of the operand itself and of its use as the transpose (the
    same stored matrix as the other GEMM's operand)."""
    M, N, K = case["M"], case["N"], case["K"]
    own = _plan(case, M, N, K, case["ab"])
    # B = W (K x N) forward; backward B = W^T (N x K). A = X (M x K) is
    # packed from its stored transpose under the plan of the same GEMM.
    flipped = (_plan(case, M, K, N, case["ab"]) if case["op"] == "B" else own) if case["trans"] else None
    return own, flipped


def _prepare_pack(case, seed):
    op = ccl.CCL_A if case["op"] == "A" else ccl.CCL_B
    rows, cols = (case["M"], case["K"]) if case["op"] == "A" else (case["K"], case["N"])
    dtype = AB[case["ab"]][1]
    own, flipped = _pack_plans(case)
    st = {"case": case, "op": op, "own": own, "flipped": flipped}
    if case["rows"] or case["op"] == "B":
        st["src"] = _source(case, seed, 1, rows, cols, WEIGHT if case["ab"] != "fp8" else 1.0, False, case["ld_pad"])
    if case["rows"]:
        st["dst"] = _buffer(own, op, dtype)
    if case["trans"]:
        st["src_t"] = st["src"] if case["op"] == "B" else _source(case, seed, 2, rows, cols, ACT, True, case["ld_pad"])
        st["dst_t"] = _buffer(flipped, op, dtype)
    if case["unpack"]:
        back = own if case["rows"] else flipped
        lay = ccl.ccl_plan_layout(back, op)
        st["out"] = torch.empty(lay.rows, lay.cols, dtype=dtype, device=DEV)
    return st


# ---- one pass ----------------------------------------------------------------

def run(state):
    return {"gemm": _run_gemm, "ffn": _run_ffn, "pack": _run_pack}[state["case"]["kind"]](state)


def _multiply(plan, a, b, c, split, alpha=1.0, beta=0.0):
    ranges, ws, ws_bytes = split
    if ranges > 1:
        ccl.ccl_gemm_splitk(plan, alpha, a, b, beta, c, ranges, ws, ws_bytes)
    elif alpha == 1.0 and beta == 0.0:
        ccl.ccl_gemm(plan, a, b, c)
    else:
        ccl.ccl_gemm_scaled(plan, alpha, a, b, beta, c)


def _run_gemm(st):
    case, plan = st["case"], st["plan"]
    ccl.ccl_pack(plan, ccl.CCL_A, st["a_src"], st["a_src"].stride(0), int(case["a_trans"]), st["a"])
    if case["b_live"]:
        ccl.ccl_pack(plan, ccl.CCL_B, st["b_src"], st["b_src"].stride(0), 0, st["b"])
    _multiply(plan, st["a"], st["b"], st["c"], (st["ranges"], st["ws"], st["ws_bytes"]), case["alpha"], case["beta"])
    if not case["unpack"]:
        return st["c"]
    ccl.ccl_unpack(plan, ccl.CCL_C, st["c"], st["out"], case["N"])
    return st["out"]


def _run_ffn(st):
    case = st["case"]
    ccl.ccl_pack(st["up"], ccl.CCL_A, st["x_src"], case["D"], 0, st["x"])
    _multiply(st["up"], st["x"], st["w_up"], st["h"], st["up_split"])
    _multiply(st["down"], st["h"], st["w_down"], st["y"], st["down_split"])
    ccl.ccl_unpack(st["down"], ccl.CCL_C, st["y"], st["out"], case["D"])
    return st["out"]


def _run_pack(st):
    case, op, got = st["case"], st["op"], {}
    if case["rows"]:
        ccl.ccl_pack(st["own"], op, st["src"], st["src"].stride(0), 0, st["dst"])
        got["packed"] = st["dst"]
    if case["trans"]:
        ccl.ccl_pack(st["flipped"], op, st["src_t"], st["src_t"].stride(0), 1, st["dst_t"])
        got["packed_transpose"] = st["dst_t"]
    if case["unpack"]:
        plan, buf = (st["own"], st["dst"]) if case["rows"] else (st["flipped"], st["dst_t"])
        ccl.ccl_unpack(plan, op, buf, st["out"], st["out"].stride(0))
        got["unpacked"] = st["out"]
    return got


# ---- what a pass cannot do without, and how exact it is ------------------------

def work(case):
    """Each input read once and each result written once. Weights arrive in
    CCL, activations as stored; intermediates are not counted."""
    if case["kind"] == "gemm":
        M, N, K, e, ec = case["M"], case["N"], case["K"], AB[case["ab"]][2], CT[case["c"]][2]
        read = (M * K + K * N) * e + (M * N * ec if case["beta"] else 0)
        return {"bytes": read + M * N * ec, "flops": 2 * M * N * K}
    if case["kind"] == "ffn":
        M, D, F = case["M"], case["D"], case["F"]
        return {"bytes": 2 * (2 * M * D + 2 * D * F), "flops": 4 * M * D * F}
    rows, cols = (case["M"], case["K"]) if case["op"] == "A" else (case["K"], case["N"])
    return {"bytes": 2 * rows * cols * AB[case["ab"]][2] * (case["rows"] + case["trans"] + case["unpack"]), "flops": 0}


def tolerance(case):
    if case["kind"] == "pack":
        return "exact"
    # Four times what was measured against exact(): 1.7e-3 for a bf16 result
    # (its rounding), 2.3e-3 where the intermediate is rounded to bf16 too,
    # 3.8e-7 for an fp32 result (fp32 sums over K = 8192).
    # "max": one unit in the last place of bf16 is at most 2^-7 of the value.
    if case["kind"] == "ffn":
        return {"rel": 1e-2, "max": 0.06}
    if case["c"] == "fp32":
        return {"rel": 1.6e-6, "max": 6e-5}
    return {"rel": 6.6e-3, "max": 0.016}


def _ccl_of(x, gr, gc, page, elem_bytes):
    """Matrix x in CCL: its gr x gc blocks one after another, each padded to
    whole pages (with zeros, as _buffer made them)."""
    R, C = x.shape
    n = (R // gr) * (C // gc)
    blocks = x.view(gr, R // gr, gc, C // gc).permute(0, 2, 1, 3).reshape(gr * gc, n)
    stride = -(-n * elem_bytes // page) * page // elem_bytes
    out = torch.zeros(gr * gc, stride, dtype=x.dtype, device=x.device)
    out[:, :n] = blocks
    return out.view(-1)


def _product64(a, b):
    """a b in 64 bits, by blocks of rows."""
    b64 = b.double()
    return torch.cat([a[r:r + 2048].double() @ b64 for r in range(0, a.shape[0], 2048)])


def exact(case, seed):
    if case["kind"] == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        a = _source(case, seed, 1, M, K, case["a_std"], case["a_trans"])
        c = _product64((a.float().t() if case["a_trans"] else a).contiguous(), _source(case, seed, 2, K, N, case["b_std"]))
        c.mul_(case["alpha"])
        if case["beta"]:
            c.add_(_normal(seed, 3, M, N, 1.0, case["c"]).double(), alpha=case["beta"])
        if case["unpack"]:
            return c
        gr, gc = ccl.ccl_plan_grid(_plan(case, M, N, K, case["ab"], case["c"]))
        return _ccl_of(c, gr, gc, case["page"], CT[case["c"]][2])
    if case["kind"] == "ffn":
        M, D, F = case["M"], case["D"], case["F"]
        h = _product64(_normal(seed, 1, M, D, ACT, "bf16"), _normal(seed, 2, D, F, WEIGHT, "bf16"))
        return _product64(h, _normal(seed, 3, F, D, WEIGHT, "bf16"))
    return None
