"""bf16 GEMM with one tile row per partition (decode batches): above the
Infinity Cache size B goes past the L2 (non-temporal loads; forced here, as the
matrices are small), below it B is cached (CCL_GEMM_STREAM_B=0). Ternary inputs,
so C equals the oracle's product exactly; whole and ragged K blocks, split-K,
every tile of one row, and every epilogue of the streaming kernels."""
import numpy as np
import pytest

import workloads as W
from oracle import gemm as OG
from oracle import layout as OL
from paper_2606_11718_amd import ccl
from tests.test_gpu_splitk import BF16, FP32, _dev_bytes, _draw, _from_dev, _to_dev, run_splitk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stream", ["1", "0"])
@pytest.mark.parametrize("tile,M,N,K,G,Gr,splits", [
    ("128x128", 128, 3072, 8 * 64 * 3, 8, 1, 1),
    ("128x128", 128, 1024, 8 * 96, 8, 1, 1),        # ragged K blocks
    ("128x128", 128, 2048, 8 * 64 * 5, 8, 1, 4),
    ("128x256", 256, 1024, 4 * 64, 4, 2, 1),        # two partition rows of one tile row each
    ("256x128", 256, 1024, 8 * 128, 8, 1, 3),
])
def test_one_tile_row(tile, M, N, K, G, Gr, splits, stream, monkeypatch):
    monkeypatch.setenv("CCL_GEMM_STREAM_B", stream)
    monkeypatch.setenv("CCL_GEMM_TILE", tile)
    monkeypatch.setenv("CCL_GEMM_STAGE_K", "64")
    A = _draw(BF16, 6100 + K, M, K, "ternary")
    B = _draw(BF16, 6101 + K, K, N, "ternary")
    run = ccl.ccl_debug_launch(ccl.ccl_plan_typed(M, N, K, G, Gr, 4096, BF16, FP32), splits)
    assert (run.kernel, run.stream_b) == ("gemm_k64_kernel", stream == "1")
    C, _ = run_splitk(A, B, M, N, K, G, Gr, BF16, FP32, splits)
    assert np.array_equal(C, OG.gemm_fp64(A, B))


@pytest.mark.parametrize("c,alpha,beta", [(BF16, 1.0, 0.0), (BF16, -0.5, 0.0), (BF16, 1.0, 2.0), (FP32, 1.0, 0.0),
                                          (FP32, 0.5, -1.0)])
@pytest.mark.parametrize("tile,M,N,K,G,Gr", [
    ("128x192", 128, 8 * 384, 8 * 128, 8, 1), ("128x192", 128, 8 * 384, 8 * 96, 8, 1),      # whole and ragged K blocks
    ("128x192", 256, 4 * 768, 4 * 64 * 5, 8, 2), ("128x192", 128, 1152, 64 * 9, 1, 1),
    ("128x320", 128, 8 * 640, 8 * 128, 8, 1), ("128x320", 128, 8 * 640, 8 * 96, 8, 1),
    ("128x320", 512, 2 * 1280, 4 * 64 * 3, 8, 4), ("128x320", 128, 1920, 64 * 7, 1, 1),
    ("128x128", 128, 8 * 256, 8 * 64, 8, 1), ("128x256", 256, 4 * 512, 4 * 192, 8, 2), ("256x128", 256, 8 * 128, 8 * 128, 8, 1),
])
def test_epilogues(tile, M, N, K, G, Gr, c, alpha, beta, monkeypatch):
    """Streamed against not streamed bit for bit, and the oracle's value."""
    rows, cols = map(int, tile.split("x"))
    monkeypatch.setenv(*(("CCL_GEMM_WIDE", str(cols)) if cols in (192, 320) else ("CCL_GEMM_TILE", tile)))
    A, B = W.draw_array(6200 + K, M, K, "ternary"), W.draw_array(6201 + K, K, N, "ternary")
    c0 = OG.decode_bf16(W.draw_array(6202, M, N, "ternary"))
    start = np.full((M, N), np.nan, dtype=np.float32) if beta == 0.0 else c0.astype(np.float32)
    bits = start.view(np.uint32) if c == FP32 else (start.view(np.uint32) >> 16).astype(np.uint16)
    got = []
    for stream in ("1", "0"):
        monkeypatch.setenv("CCL_GEMM_STREAM_B", stream)
        plan = ccl.ccl_plan_typed(M, N, K, G, Gr, 4096, BF16, c)
        run = ccl.ccl_debug_launch(plan, reads_c=int(beta != 0.0))
        assert (run.kernel, run.tile_rows, run.tile_cols, run.stream_b) == ("gemm_k64_kernel", rows, cols, stream == "1")
        assert run.ragged == (K // (G // Gr) % 64 != 0)
        print(f"stream_b {tile} {M}x{N}x{K} c={c} alpha={alpha} beta={beta} stream={stream}", flush=True)
        gr, gc = ccl.ccl_plan_grid(plan)
        Ac, Bc = (_dev_bytes(ccl.ccl_plan_layout(plan, op).total_bytes) for op in (ccl.CCL_A, ccl.CCL_B))
        ccl.ccl_pack(plan, ccl.CCL_A, _to_dev(A), K, 0, Ac)
        ccl.ccl_pack(plan, ccl.CCL_B, _to_dev(B), N, 0, Bc)
        Cc = _to_dev(OL.pack(bits, gr, gc, 4096))
        ccl.ccl_gemm_scaled(plan, alpha, Ac, Bc, beta, Cc)
        got.append(OL.unpack(_from_dev(Cc, np.uint32 if c == FP32 else np.uint16), M, N, gr, gc, 4096))
    assert np.array_equal(*got)
    want = OG.gemm_scaled_fp64(OG.decode_bf16(A), OG.decode_bf16(B), c0, alpha, beta).astype(np.float32)
    if c == FP32:
        assert np.array_equal(got[0].view(np.float32), want)
    else:
        assert np.array_equal(OG.decode_bf16(got[0]), OG.decode_bf16(W.round_to_bf16_bits(want)))
