"""bf16 GEMM with 64-K stages on operands of 2 GiB and more (the far form moves
its descriptors with the stages): the 32-K kernel's C bit for bit, forced at
small sizes over step counts, K blocks and split-K ranges, and at its own size
on both operands."""
import numpy as np
import pytest

import workloads as W
from oracle import gemm as OG
from paper_2606_11718_amd import ccl
from tests.test_gpu_gemm_ragged import _gemm
from tests.test_gpu_splitk import BF16, FP32, _draw, run_splitk

pytestmark = pytest.mark.gpu


def _form(monkeypatch, far, M, N, K, G, Gr, splits=1):
    monkeypatch.setenv("CCL_GEMM_FAR" if far else "CCL_GEMM_STAGE_K", "1" if far else "32")
    monkeypatch.delenv("CCL_GEMM_STAGE_K" if far else "CCL_GEMM_FAR", raising=False)
    run = ccl.ccl_debug_launch(ccl.ccl_plan(M, N, K, G, Gr, 4096), splits)
    assert (run.kernel, run.far) == (("gemm_k64_kernel", True) if far else ("gemm_kernel", False))


@pytest.mark.parametrize("stream", ["0", "1"])
@pytest.mark.parametrize("tile", ["256x128", "128x256", "128x128"])
@pytest.mark.parametrize("G,Gr,M,N,K", [
    (1, 1, 256, 256, 64), (1, 1, 256, 256, 128), (1, 1, 256, 256, 192), (1, 1, 256, 256, 256),
    (1, 1, 256, 256, 64 * 9), (8, 1, 256, 2048, 8 * 64), (8, 2, 512, 1024, 4 * 128), (8, 8, 2048, 256, 8 * 192)])
def test_equals_32k_stages(stream, tile, G, Gr, M, N, K, monkeypatch):
    monkeypatch.setenv("CCL_GEMM_TILE", tile)
    monkeypatch.setenv("CCL_GEMM_STREAM_B", stream)
    A = W.draw_array(9500 + K, M, K, "normal", 1.0)
    B = W.draw_array(9501 + K, K, N, "normal", 0.05)
    got = []
    for far in (True, False):
        _form(monkeypatch, far, M, N, K, G, Gr)
        got.append(_gemm(A, B, M, N, K, G, Gr))
    assert np.array_equal(*got)
    assert OG.within_tolerance(OG.errors(OG.decode_bf16(got[0]), OG.gemm_fp64(A, B)))


@pytest.mark.parametrize("M,N,K,G,Gr,splits", [(256, 1024, 8 * 64 * 5, 8, 1, 4), (1024, 256, 8 * 64 * 3, 8, 8, 5)])
def test_splitk(M, N, K, G, Gr, splits, monkeypatch):
    A, B = _draw(BF16, 9600 + K, M, K), _draw(BF16, 9601 + K, K, N, "normal", 0.05)
    got = []
    for far in (True, False):
        _form(monkeypatch, far, M, N, K, G, Gr, splits)
        got.append(run_splitk(A, B, M, N, K, G, Gr, BF16, FP32, splits)[0])
    assert np.array_equal(*got)


@pytest.mark.parametrize("M,N,K,G", [(128, 131072, 8192, 1), (131072, 1024, 9728, 8)])
def test_two_gib_operand(M, N, K, G, monkeypatch):
    """B in one block of 2 GiB, and A in 8 blocks of more in all; no override."""
    torch = __import__("torch")
    gen = torch.Generator(device="cuda").manual_seed(M + K)
    print(f"far {M}x{N}x{K}", flush=True)
    out = []
    for env in (None, "32"):
        if env:
            monkeypatch.setenv("CCL_GEMM_STAGE_K", env)
        plan = ccl.ccl_plan(M, N, K, G, 1, 4096)
        assert ccl.ccl_debug_launch(plan).far == (env is None)
        la, lb, lc = (ccl.ccl_plan_layout(plan, op) for op in (ccl.CCL_A, ccl.CCL_B, ccl.CCL_C))
        if not out:
            assert max(la.total_bytes, lb.total_bytes) >= 1 << 31
            A = torch.empty(la.total_bytes // 2, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
            B = torch.empty(lb.total_bytes // 2, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
        C = torch.zeros(lc.total_bytes // 2, dtype=torch.int16, device="cuda")
        ccl.ccl_gemm(plan, A, B, C)
        torch.cuda.synchronize()
        out.append(C)
    assert bool(out[0].any()) and torch.equal(*out)
