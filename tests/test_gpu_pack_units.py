"""Pack and unpack around the sizes where a thread's share changes (1, 2 or 4
units of 16 bytes, by the units per strip that 2048 workgroups hold): the largest
of each and the next one, with whole and overlapping last units and a wide
leading dimension. Bytes against the oracle's layout, and back."""
import numpy as np
import pytest

from oracle import layout as OL
from paper_2606_11718_amd import ccl
from tests.helpers import dev_full, from_dev, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("G,M,K", [
    (1, 128, 16), (1, 1536, 2048), (1, 1536, 2056), (1, 2048, 2048), (1, 2048, 2056), (1, 2048, 4096), (1, 2048, 4104), (1, 2048, 2042),
    (8, 128, 16384), (8, 128, 8 * 2052), (8, 2048, 8 * 260), (8, 4096, 8 * 260)])
def test_pack_and_back(G, M, K, pad):
    plan = ccl.ccl_plan(M, 128 * G, K, G, 1, 4096)
    print(f"pack units G={G} {M}x{K} pad={pad}", flush=True)
    wide = np.random.default_rng(9400 + M + K).integers(0, 1 << 16, (M, K + pad), dtype=np.uint16)
    X = np.ascontiguousarray(wide[:, :K])
    lay = ccl.ccl_plan_layout(plan, ccl.CCL_A)
    src, dst, back = to_dev(wide), dev_full(lay.total_bytes // 2), dev_full(M * (K + pad))
    canary = from_dev(back).copy()
    ccl.ccl_pack(plan, ccl.CCL_A, src, K + pad, 0, dst)
    ccl.ccl_unpack(plan, ccl.CCL_A, dst, back, K + pad)
    packed = from_dev(dst)
    assert np.array_equal(packed, OL.pack_reshape(X, 1, G, 4096, int(canary[0])))
    got = from_dev(back).reshape(M, K + pad)
    assert np.array_equal(got[:, :K], X)
    assert np.all(got[:, K:] == canary[0])
