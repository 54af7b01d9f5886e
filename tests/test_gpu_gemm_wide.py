"""bf16 GEMM on 128x192 and 128x320 tiles (CCL_GEMM_WIDE=192|320 takes them
wherever they exist, 0 the 128- and 256-wide ones). Plain C against the other tiles bit for bit (the
same MFMAs in the same order, at every K) on normal inputs; scaled, fp32 and
read C against the oracle, exact on ternary inputs."""
import numpy as np
import pytest

import workloads as W
from oracle import gemm as OG
from oracle import layout as OL
from paper_2606_11718_amd import ccl
from tests.test_gpu_gemm_ragged import _gemm
from tests.test_gpu_splitk import BF16, FP32, _dev_bytes, _from_dev, _to_dev

pytestmark = pytest.mark.gpu


def _check_tile(wide, plan, operands=0):
    """The launch runs 128 x wide tiles ("0": others)."""
    run = ccl.ccl_debug_launch(plan, operands=operands)
    assert (run.kernel, run.tile_cols) == ("gemm_k64_kernel", int(wide)) if wide != "0" else run.tile_cols in (128, 256)


@pytest.mark.parametrize("wide,G,Gr,M,N,K", [("192",) + c for c in [
    (1, 1, 128, 384, 64), (1, 1, 128, 384, 64 * 3), (1, 1, 128, 384, 64 * 4), (1, 1, 128, 384, 64 * 7),
    (1, 1, 128, 384, 64 * 8), (1, 1, 128, 384, 64 * 13), (1, 1, 256, 768, 96), (1, 1, 128, 384, 32 * 15),
    (8, 2, 2048, 1536, 4 * 128),        # 32 tiles per XCD, whole K blocks
    (8, 2, 512, 3072, 4 * 160),         # A: blocks of 5 steps, B: 10
    (8, 8, 2048, 384, 8 * 96),          # B: blocks of 3 steps
    (8, 1, 128, 8 * 1152, 8 * 64),      # one tile row, 6 tile columns
    (4, 2, 2560, 768, 256),             # 10 tile rows: a whole raster group and a short one
]] + [("320",) + c for c in [
    (1, 1, 128, 640, 64), (1, 1, 128, 640, 64 * 2), (1, 1, 128, 640, 64 * 3), (1, 1, 128, 640, 64 * 4),
    (1, 1, 128, 640, 64 * 5), (1, 1, 128, 640, 64 * 8), (1, 1, 256, 640, 96), (1, 1, 128, 640, 32 * 15),
    (8, 1, 1920, 5120, 1792),           # 30 tiles per XCD, K blocks of 7 steps
    (8, 2, 512, 2560, 4 * 160), (8, 8, 2048, 640, 8 * 96), (8, 1, 128, 8 * 1280, 8 * 64),
]])
def test_equals_other_tiles(wide, G, Gr, M, N, K, monkeypatch):
    A = W.draw_array(9100 + K, M, K, "normal", 1.0)
    B = W.draw_array(9101 + K, K, N, "normal", 0.05)
    got = {}
    for n in ("0", wide):
        monkeypatch.setenv("CCL_GEMM_WIDE", n)
        _check_tile(n, ccl.ccl_plan(M, N, K, G, Gr, 4096))
        got[n] = _gemm(A, B, M, N, K, G, Gr)
    assert np.array_equal(got["0"], got[wide])
    assert OG.within_tolerance(OG.errors(OG.decode_bf16(got[wide]), OG.gemm_fp64(A, B)))


@pytest.mark.parametrize("wide", ["192", "320"])
@pytest.mark.parametrize("c,alpha,beta", [(BF16, -0.5, 0.0), (BF16, 1.0, 2.0), (FP32, 1.0, 0.0),
                                          (FP32, 2.0, 0.0), (FP32, 0.5, -1.0)])
def test_epilogues(wide, c, alpha, beta, monkeypatch):
    monkeypatch.setenv("CCL_GEMM_WIDE", wide)
    M, N, K, G, Gr = 512, 4 * int(wide) * 2, 512, 4, 2
    A, B = W.draw_array(9200, M, K, "ternary"), W.draw_array(9201, K, N, "ternary")
    C0 = W.draw_array(9202, M, N, "ternary")
    plan = ccl.ccl_plan_typed(M, N, K, G, Gr, 4096, BF16, c)
    _check_tile(wide, plan)
    gr, gc = ccl.ccl_plan_grid(plan)
    print(f"wide epilogue {wide} c={c} alpha={alpha} beta={beta}", flush=True)
    Ac, Bc = (_dev_bytes(ccl.ccl_plan_layout(plan, op).total_bytes) for op in (ccl.CCL_A, ccl.CCL_B))
    ccl.ccl_pack(plan, ccl.CCL_A, _to_dev(A), K, 0, Ac)
    ccl.ccl_pack(plan, ccl.CCL_B, _to_dev(B), N, 0, Bc)
    c0 = OG.decode_bf16(C0)
    start = np.full((M, N), np.nan, dtype=np.float32) if beta == 0.0 else c0.astype(np.float32)
    bits = start.view(np.uint32) if c == FP32 else (start.view(np.uint32) >> 16).astype(np.uint16)
    Cc = _to_dev(OL.pack(bits, gr, gc, 4096))
    ccl.ccl_gemm_scaled(plan, alpha, Ac, Bc, beta, Cc)
    want = OG.gemm_scaled_fp64(OG.decode_bf16(A), OG.decode_bf16(B), c0, alpha, beta).astype(np.float32)
    got = OL.unpack(_from_dev(Cc, np.uint32 if c == FP32 else np.uint16), M, N, gr, gc, 4096)
    if c == FP32:
        assert np.array_equal(got.view(np.float32), want)
    else:
        assert np.array_equal(OG.decode_bf16(got), OG.decode_bf16(W.round_to_bf16_bits(want)))


@pytest.mark.parametrize("wide", ["192", "320"])
def test_rowmajor(wide, monkeypatch):
    """Row-major operands under the XCD-aware map (one K block)."""
    monkeypatch.setenv("CCL_GEMM_WIDE", wide)
    M, N, K = 512, 4 * int(wide) * 2, 320
    A, B = W.draw_array(9300, M, K, "ternary"), W.draw_array(9301, K, N, "ternary")
    plan = ccl.ccl_plan(M, N, K, 4, 2, 4096)
    _check_tile(wide, plan, operands=2)
    C = _dev_bytes(M * N * 2)
    ccl.ccl_gemm_rowmajor(plan, _to_dev(A), _to_dev(B), C, 1)
    got = OG.decode_bf16(_from_dev(C, np.uint16).reshape(M, N))
    assert np.array_equal(got, OG.decode_bf16(W.round_to_bf16_bits(OG.gemm_fp64(A, B).astype(np.float32))))
