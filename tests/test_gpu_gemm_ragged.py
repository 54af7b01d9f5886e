"""bf16 GEMM tiles below 256x256 on K blocks and K ranges that are odd
multiples of 32: the 64-K stages (CCL_GEMM_STAGE_K=64, as plans do not take
them everywhere) then straddle K blocks, and the last one may be half empty.
Against the 32-K kernel (the same MFMAs in the same order, so bit for bit) and
the oracle. K blocks of one 32-K step have the 32-K kernel only."""
import numpy as np
import pytest

import workloads as W
from oracle import gemm as OG
from oracle import layout as OL
from paper_2606_11718_amd import ccl
from tests.helpers import from_dev, to_dev
from tests.test_gpu_splitk import BF16, FP32, _draw, run_splitk

pytestmark = pytest.mark.gpu

NAN = 0x7FC0


def _gemm(A, B, M, N, K, G, Gr):
    """The GEMM on packed operands whose padding holds NaN, and 512 NaN on
    either side of both operands."""
    plan = ccl.ccl_plan(M, N, K, G, Gr, 4096)
    gr, gc = ccl.ccl_plan_grid(plan)
    print(f"ragged gemm {M}x{N}x{K} grid {gr}x{gc} {ccl.ccl_debug_gemm_config(plan)}", flush=True)
    guard = np.full(512, NAN, dtype=np.uint16)
    Ad, Bd = (to_dev(np.concatenate([guard, OL.pack_reshape(X, gr, gc, 4096, NAN), guard])) for X in (A, B))
    lc = ccl.ccl_plan_layout(plan, ccl.CCL_C)
    Cd = to_dev(np.full(lc.total_bytes // 2, NAN, dtype=np.uint16))
    ccl.ccl_gemm(plan, Ad.data_ptr() + 1024, Bd.data_ptr() + 1024, Cd)
    return OL.unpack(from_dev(Cd), M, N, gr, gc, 4096)


def _stages(monkeypatch, k, M, N, K, G, Gr, splits=1):
    """Plans with k-K stages from here on; checks that they run."""
    monkeypatch.setenv("CCL_GEMM_STAGE_K", str(k))
    run = ccl.ccl_debug_launch(ccl.ccl_plan(M, N, K, G, Gr, 4096), splits)
    one_step = min(K // Gr, K // (G // Gr)) < 64
    assert (run.kernel, run.ragged) == (("gemm_kernel", False) if k == 32 or one_step else ("gemm_k64_kernel", True))


@pytest.mark.parametrize("tile", ["256x128", "128x256", "128x128"])
@pytest.mark.parametrize("G,Gr,M,N,K", [
    (1, 1, 256, 256, 32), (1, 1, 256, 256, 96), (1, 1, 256, 256, 32 * 7), (1, 1, 256, 256, 32 * 19),
    (8, 1, 256, 2048, 8 * 32),          # A: 8 blocks of one 32-K step
    (8, 1, 256, 2048, 8 * 96),          # A: blocks of 3 steps
    (8, 8, 2048, 256, 8 * 32 * 7),      # B: blocks of 7 steps
    (4, 2, 512, 512, 2 * 32 * 13),      # both: blocks of 13 steps
    (8, 2, 512, 1024, 4 * 160),         # A: 5 steps, B: 10
])
def test_equals_32k_stages(tile, G, Gr, M, N, K, monkeypatch):
    monkeypatch.setenv("CCL_GEMM_TILE", tile)
    A = W.draw_array(5500 + K, M, K, "normal", 1.0)
    B = W.draw_array(5501 + K, K, N, "normal", 0.05)
    _stages(monkeypatch, 64, M, N, K, G, Gr)
    c64 = _gemm(A, B, M, N, K, G, Gr)
    _stages(monkeypatch, 32, M, N, K, G, Gr)
    c32 = _gemm(A, B, M, N, K, G, Gr)
    assert np.array_equal(c64, c32)
    assert OG.within_tolerance(OG.errors(OG.decode_bf16(c64), OG.gemm_fp64(A, B)))


@pytest.mark.parametrize("M,N,K,G,Gr,splits", [
    (256, 1024, 8 * 32 * 5, 8, 1, 3),       # 40 steps in ranges of 14, 14, 12
    (256, 1024, 8 * 32 * 5, 8, 1, 6),       # ranges of 7 steps start off the 64-K grid
    (1024, 256, 8 * 32 * 3, 8, 8, 5),       # 24 steps in ranges of 5, the last 4
    (768, 2048, 4096, 8, 1, 3),             # whole 64-K blocks, ranges of 43 steps
])
def test_splitk_equals_32k_stages(M, N, K, G, Gr, splits, monkeypatch):
    A = _draw(BF16, 5600 + M + K, M, K)
    B = _draw(BF16, 5700 + N + K, K, N, "normal", 0.05)
    _stages(monkeypatch, 64, M, N, K, G, Gr, splits)
    C64, r64 = run_splitk(A, B, M, N, K, G, Gr, BF16, FP32, splits)
    _stages(monkeypatch, 32, M, N, K, G, Gr, splits)
    C32, r32 = run_splitk(A, B, M, N, K, G, Gr, BF16, FP32, splits)
    assert r64 == r32
    assert np.array_equal(C64, C32)
    assert OG.errors(C64, OG.gemm_fp64(A, B))["rel_fro"] <= 1e-4
