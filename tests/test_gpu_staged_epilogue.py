"""The LDS-staged epilogues of a scaled, an fp32 and a read C, for every tile
of the bf16 and fp8 kernels. Ternary A, B and C0 and power-of-two scalars
keep alpha acc + beta c exact in fp32, so C must equal the oracle's value
(rounded to nearest even for a bf16 C) bit for bit. Two tiles per partition
side and several partitions, so a misplaced row or column shows."""
import numpy as np
import pytest

import workloads as W
from oracle import gemm as OG
from oracle import layout as OL
from paper_2606_11718_amd import ccl
from tests.test_gpu_splitk import _dev_bytes, _from_dev, _to_dev

pytestmark = pytest.mark.gpu

BF16, FP8, FP32 = ccl.CCL_DT_BF16, ccl.CCL_DT_FP8_E4M3, ccl.CCL_DT_FP32


@pytest.mark.parametrize("tile", ["256x256", "256x128", "128x256", "128x128"])
@pytest.mark.parametrize("ab", [BF16, FP8])
@pytest.mark.parametrize("c,alpha,beta", [(BF16, -0.5, 0.0), (BF16, 1.0, 2.0), (FP32, 1.0, 0.0),
                                          (FP32, 2.0, 0.0), (FP32, 0.5, -1.0)])
def test_every_tile(tile, ab, c, alpha, beta, monkeypatch):
    monkeypatch.setenv("CCL_GEMM_TILE", tile)
    M, N, K, G, Gr = 1024, 1024, 512, 4, 2
    draw, dec = (W.draw_array, OG.decode_bf16) if ab == BF16 else (W.draw_array_fp8, OG.decode_fp8_e4m3)
    A, B = draw(8100, M, K, "ternary"), draw(8101, K, N, "ternary")
    C0 = W.draw_array(8102, M, N, "ternary")
    plan = ccl.ccl_plan_typed(M, N, K, G, Gr, 4096, ab, c)
    gr, gc = ccl.ccl_plan_grid(plan)
    print(f"staged epilogue {tile} ab={ab} c={c} alpha={alpha} beta={beta}", flush=True)
    la, lb = (ccl.ccl_plan_layout(plan, op) for op in (ccl.CCL_A, ccl.CCL_B))
    Ac, Bc = _dev_bytes(la.total_bytes), _dev_bytes(lb.total_bytes)
    ccl.ccl_pack(plan, ccl.CCL_A, _to_dev(A), K, 0, Ac)
    ccl.ccl_pack(plan, ccl.CCL_B, _to_dev(B), N, 0, Bc)
    c0 = OG.decode_bf16(C0)
    if beta == 0.0:                                   # C must not be read: start from NaN
        start = np.full((M, N), np.nan, dtype=np.float32)
    else:
        start = c0.astype(np.float32)
    bits = start.view(np.uint32) if c == FP32 else (start.view(np.uint32) >> 16).astype(np.uint16)
    Cc = _to_dev(OL.pack(bits, gr, gc, 4096))
    ccl.ccl_gemm_scaled(plan, alpha, Ac, Bc, beta, Cc)
    want = OG.gemm_scaled_fp64(dec(A), dec(B), c0, alpha, beta).astype(np.float32)
    got = OL.unpack(_from_dev(Cc, np.uint32 if c == FP32 else np.uint16), M, N, gr, gc, 4096)
    if c == FP32:
        assert np.array_equal(got.view(np.float32), want)
    else:
        assert np.array_equal(OG.decode_bf16(got), OG.decode_bf16(W.round_to_bf16_bits(want)))
