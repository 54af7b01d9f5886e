"""bf16 GEMM with one tile row per partition (decode batches): above the
Infinity Cache size B goes past the L2 (non-temporal loads; forced here, as the
matrices are small), below it B is cached (CCL_GEMM_STREAM_B=0). Ternary inputs, so C equals the oracle's product
exactly; whole and ragged K blocks, split-K, every tile of one row."""
import numpy as np
import pytest

from oracle import gemm as OG
from paper_2606_11718_amd import ccl
from tests.test_gpu_splitk import BF16, FP32, _draw, run_splitk

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
    A = _draw(BF16, 6100 + K, M, K, "ternary")
    B = _draw(BF16, 6101 + K, K, N, "ternary")
    C, _ = run_splitk(A, B, M, N, K, G, Gr, BF16, FP32, splits)
    assert np.array_equal(C, OG.gemm_fp64(A, B))
