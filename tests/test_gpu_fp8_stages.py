"""fp8 GEMM on 128-K stages (tiles below 256x256): step counts that stop in
the prologue, the rounds and the tail of its ring of 3 or 4 stages, CCL K
blocks, and split-K ranges. Ternary inputs: every sum is an exact integer in
fp32, so C must equal the oracle's product bit for bit."""
import numpy as np
import pytest

import workloads as W
from oracle import gemm as OG
from paper_2606_11718_amd import ccl
from tests.test_gpu_fp8 import run_fp8
from tests.test_gpu_splitk import run_splitk

pytestmark = pytest.mark.gpu

FP8, FP32 = ccl.CCL_DT_FP8_E4M3, ccl.CCL_DT_FP32


def _check_kernel(M, N, K, G, Gr, tile, monkeypatch, splits=1):
    monkeypatch.setenv("CCL_GEMM_TILE", tile)
    run = ccl.ccl_debug_launch(ccl.ccl_plan_typed(M, N, K, G, Gr, 4096, FP8, FP32), splits)
    assert (run.kernel, f"{run.tile_rows}x{run.tile_cols}") == ("gemm_fp8s_kernel", tile)
    monkeypatch.delenv("CCL_GEMM_TILE")


def _inputs(M, N, K):
    A = W.draw_array_fp8(7000 + M + K, M, K, "ternary")
    B = W.draw_array_fp8(7100 + N + K, K, N, "ternary")
    return A, B, OG.gemm_fp64(OG.decode_fp8_e4m3(A), OG.decode_fp8_e4m3(B))


@pytest.mark.parametrize("tile", ["128x128", "256x128", "128x256"])
@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 8, 9, 11, 13])
def test_step_counts(tile, steps, monkeypatch):
    M, N, K = 256, 256, 128 * steps
    _check_kernel(M, N, K, 1, 1, tile, monkeypatch)
    A, B, ref = _inputs(M, N, K)
    C = run_fp8(A, B, M, N, K, 1, 1, c_type=FP32, tile=tile)[0]
    assert np.array_equal(C, ref)


@pytest.mark.parametrize("M,N,K,G,Gr,tile", [
    (512, 1024, 1024, 8, 2, "256x128"),      # K blocks of 2 steps (A) and 4 (B)
    (1024, 256, 3072, 8, 4, "128x128"),      # 12 and 6 steps
    (256, 512, 768, 4, 2, "128x256"),        # 3 steps per block on both
])
def test_k_blocks(M, N, K, G, Gr, tile, monkeypatch):
    _check_kernel(M, N, K, G, Gr, tile, monkeypatch)
    A, B, ref = _inputs(M, N, K)
    C = run_fp8(A, B, M, N, K, G, Gr, c_type=FP32, tile=tile)[0]
    assert np.array_equal(C, ref)


@pytest.mark.parametrize("tile", ["128x128", "256x128", "128x256"])
@pytest.mark.parametrize("splits", [2, 3, 4, 5])    # ranges of 12, 8, 6 and 5 stages, the last of 5 shorter
def test_splitk(tile, splits, monkeypatch):
    M, N, K, G, Gr = 512, 1024, 3072, 8, 2
    _check_kernel(M, N, K, G, Gr, tile, monkeypatch, splits)
    monkeypatch.setenv("CCL_GEMM_TILE", tile)
    A, B, ref = _inputs(M, N, K)
    C, _ = run_splitk(A, B, M, N, K, G, Gr, FP8, FP32, splits)
    assert np.array_equal(C, ref)
