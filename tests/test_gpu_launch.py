"""ccl_gemm's own launch on the GPU where it differs from the plan's tile
(128x192 and 128x320): workgroups on the owners' XCDs, and a timeline launch
with ccl_gemm's C bit for bit."""
import numpy as np
import pytest

import workloads as W
from oracle import plan as OP
from paper_2606_11718_amd import ccl
from tests.helpers import dev_full, from_dev, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [("192", 4096, 1536, 2048, 8, 2), ("192", 2560, 768, 256, 4, 2), ("320", 1920, 5120, 1792, 8, 1),
          ("320", 1408, 640, 512, 1, 1)]


@pytest.mark.parametrize("wide,M,N,K,G,Gr", SHAPES)
def test_dispatch(wide, M, N, K, G, Gr, monkeypatch):
    torch = __import__("torch")
    monkeypatch.setenv("CCL_GEMM_WIDE", wide)
    plan = ccl.ccl_plan(M, N, K, G, Gr, 4096)
    run = ccl.ccl_debug_launch(plan)
    assert run.tile_cols == int(wide)
    out = torch.full((4 * run.workgroups,), -7, dtype=torch.int32, device="cuda")
    ccl.ccl_debug_launch_dispatch(plan, out)
    rec = out.cpu().numpy().reshape(run.workgroups, 4)
    rot = (rec[:, 0] - np.arange(run.workgroups)) % 8
    assert len(set(rot.tolist())) == 1
    live = rec[rec[:, 1] >= 0]
    assert len({(a, b) for a, b in live[:, 1:3]}) == len(live) == (M // 128) * (N // int(wide))
    for wg, (xcd, ti, tj, owner) in enumerate(rec):
        assert (wg % 8, ti, tj) == ccl.ccl_debug_launch_tile_of_wg(plan, wg)
        if ti >= 0:
            assert owner == OP.owner(ti, tj * int(wide) // 128, M, N, Gr, G // Gr)
            assert (xcd - rot[0]) % 8 in OP.xcds_of_chiplet(owner, G)


@pytest.mark.parametrize("wide,M,N,K,G,Gr", SHAPES)
def test_timeline(wide, M, N, K, G, Gr, monkeypatch):
    torch = __import__("torch")
    monkeypatch.setenv("CCL_GEMM_WIDE", wide)
    plan = ccl.ccl_plan(M, N, K, G, Gr, 4096)
    run = ccl.ccl_debug_launch(plan)
    assert run.tile_cols == int(wide)
    la, lb, lc = (ccl.ccl_plan_layout(plan, op) for op in (ccl.CCL_A, ccl.CCL_B, ccl.CCL_C))
    A = to_dev(W.draw_array(71, 1, la.total_bytes // 2, "normal", 1.0)[0])
    B = to_dev(W.draw_array(72, 1, lb.total_bytes // 2, "normal", 0.05)[0])
    C1, C2 = dev_full(lc.total_bytes // 2), dev_full(lc.total_bytes // 2)
    tl = torch.zeros(run.workgroups * run.waves * 8, dtype=torch.int64, device="cuda")
    with pytest.raises(RuntimeError, match="timeline smaller"):
        ccl.ccl_debug_launch_timeline(plan, A, B, C2, tl, tl.numel() * 8 - 8)
    ccl.ccl_gemm(plan, A, B, C1)
    ccl.ccl_debug_launch_timeline(plan, A, B, C2, tl, tl.numel() * 8)
    assert np.array_equal(from_dev(C1), from_dev(C2))
    rec = tl.cpu().numpy().reshape(run.workgroups, run.waves, 8)
    live = np.array([ccl.ccl_debug_launch_tile_of_wg(plan, w)[1] >= 0 for w in range(run.workgroups)])
    assert np.all(rec[~live] == 0) and np.all(rec[live][:, :, 0] > 0)
    assert np.all(np.diff(rec[live][:, :, 0:4], axis=2) >= 0)
    assert np.all(rec[live][:, :, 5] > rec[live][:, :, 4])
