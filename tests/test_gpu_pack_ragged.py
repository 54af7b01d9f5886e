"""Packs and unpacks off the 16-byte grid: block rows that are no whole number
of 16-byte units (their last unit overlaps the one before), rows shorter than
one unit, odd leading dimensions, buffers at odd element offsets, and stored
transposes whose blocks are multiples of a thread's block only, or of
nothing. Bit-exact against the oracle's map; what lies around the written
bytes must keep its canary."""
import numpy as np
import pytest

from oracle import layout as OL
from paper_2606_11718_amd import ccl
from tests.helpers import torch_mod

pytestmark = pytest.mark.gpu

DT = {1: (ccl.CCL_DT_FP8_E4M3, ccl.CCL_DT_BF16, np.uint8), 2: (ccl.CCL_DT_BF16, ccl.CCL_DT_BF16, np.uint16),
      4: (ccl.CCL_DT_FP32, ccl.CCL_DT_FP32, np.uint32)}
CANARY = 0xA5


def _dev(host: np.ndarray, offset: int):
    """host's bytes on the GPU, `offset` bytes into a canary-filled buffer."""
    torch = torch_mod()
    raw = np.ascontiguousarray(host).view(np.uint8).reshape(-1)
    buf = torch.full((raw.size + offset + 64,), CANARY, dtype=torch.uint8, device="cuda")
    buf[offset:offset + raw.size] = torch.from_numpy(raw).to("cuda")
    return buf


def _check(e, M, N, K, G, Gr, op, trans, ld_extra, src_off, dst_off, unpack):
    torch = torch_mod()
    ab, c, dt = DT[e]
    plan = ccl.ccl_plan_typed(M, N, K, G, Gr, 4096, ab, c)
    gr, gc = ccl.ccl_plan_grid(plan)
    code = {"A": ccl.CCL_A, "B": ccl.CCL_B}[op]
    lay = ccl.ccl_plan_layout(plan, code)
    R, C = lay.rows, lay.cols
    X = np.random.default_rng(R * 31 + C).integers(0, 256, size=(R, C * e), dtype=np.uint8).view(dt)
    stored = np.ascontiguousarray(X.T) if trans else X
    ld = stored.shape[1] + ld_extra
    wide = np.zeros((stored.shape[0], ld), dtype=dt)
    wide[:, :stored.shape[1]] = stored
    print(f"ragged pack {op} {R}x{C} e={e} grid {gr}x{gc} trans={trans} ld={ld} off={src_off},{dst_off}", flush=True)
    src = _dev(wide, src_off * e)
    dst = torch.full((lay.total_bytes + dst_off * e + 64,), CANARY, dtype=torch.uint8, device="cuda")
    ccl.ccl_pack(plan, code, src.data_ptr() + src_off * e, ld, int(trans), dst.data_ptr() + dst_off * e)
    torch.cuda.synchronize()
    got = dst.cpu().numpy()
    ref = np.ascontiguousarray(OL.pack_reshape(X, gr, gc, 4096)).view(np.uint8).reshape(-1)
    body = got[dst_off * e:dst_off * e + lay.total_bytes].reshape(gr * gc, -1)
    n = lay.strip_bytes
    assert np.array_equal(body[:, :n], ref.reshape(gr * gc, -1)[:, :n])
    assert np.all(body[:, n:] == CANARY)
    assert np.all(got[:dst_off * e] == CANARY) and np.all(got[dst_off * e + lay.total_bytes:] == CANARY)
    if unpack:
        ldo = C + ld_extra
        out = torch.full((R * ldo * e + src_off * e + 64,), CANARY, dtype=torch.uint8, device="cuda")
        ccl.ccl_unpack(plan, code, dst.data_ptr() + dst_off * e, out.data_ptr() + src_off * e, ldo)
        torch.cuda.synchronize()
        flat = out.cpu().numpy()
        back = flat[src_off * e:src_off * e + R * ldo * e].reshape(R, ldo * e)
        assert np.array_equal(back[:, :C * e], X.view(np.uint8).reshape(R, C * e))
        assert np.all(back[:, C * e:] == CANARY)
        assert np.all(flat[:src_off * e] == CANARY) and np.all(flat[src_off * e + R * ldo * e:] == CANARY)


@pytest.mark.parametrize("e", [1, 2, 4])
@pytest.mark.parametrize("K,ld_extra,src_off,dst_off", [
    (8 * 3, 0, 0, 0),           # 3-element block rows: one element per unit (fp32: 12 bytes)
    (8 * 16, 1, 0, 0),          # whole units, odd leading dimension
    (8 * 17, 0, 0, 0),          # one element over a unit (fp8), last unit overlaps
    (8 * 31, 3, 1, 0),
    (8 * 64, 0, 0, 3),          # aligned rows into an odd element offset
    (8 * 101, 5, 3, 1),
])
def test_row_major(e, K, ld_extra, src_off, dst_off):
    _check(e, 384, 1024, K, 8, 1, "A", False, ld_extra, src_off, dst_off, True)


@pytest.mark.parametrize("e", [1, 2, 4])
@pytest.mark.parametrize("M,N,K,G,Gr,op,ld_extra,src_off,dst_off", [
    (384, 1024, 8 * 16, 8, 1, "A", 0, 0, 0),     # 16-column blocks: within a wave's block
    (384, 1024, 8 * 48, 8, 1, "A", 0, 0, 0),     # 48-column blocks straddle waves
    (384, 1024, 8 * 208, 8, 1, "A", 16, 0, 0),   # several waves, the last partly idle
    (384, 1024, 8 * 208, 8, 1, "A", 1, 1, 1),    # the same off the 16-byte grid
    (512, 512, 4 * 80, 4, 2, "B", 3, 0, 0),      # 160-row blocks (B splits K by rows)
    (384, 1024, 8 * 13, 8, 1, "A", 0, 0, 0),     # 13-column blocks: element tiles
    (384, 1024, 8 * 73, 8, 1, "A", 5, 3, 1),
])
def test_stored_transpose(e, M, N, K, G, Gr, op, ld_extra, src_off, dst_off):
    _check(e, M, N, K, G, Gr, op, True, ld_extra, src_off, dst_off, False)


@pytest.mark.parametrize("e,M,K,G", [
    (1, 1024, 8 * 64, 8), (1, 8 * 192, 832, 1),       # fp8, sides of 64 mod 128: LDS tiles
    (1, 2048, 8 * 576, 8), (1, 2048, 4544, 1),        # above 8 MiB: with and without 8 | tile columns
    (1, 1024, 8 * 48, 8), (1, 4096, 8 * 48, 8),       # ragged blocks of few and of more elements
    (2, 1024, 8 * 24, 8), (2, 1024, 8 * 40, 8),
    (1, 768, 8 * 37, 8), (2, 1024, 8 * 111, 8), (4, 1024, 8 * 113, 8),   # neither: 917504 elements the most
])
def test_stored_transpose_by_size(e, M, K, G):
    """Either side of the sizes where one kernel hands over to another."""
    _check(e, -(-M // 128) * 128, 1024, K, G, 1, "A", True, 0, 0, 0, False)


def test_stored_transpose_of_more_than_65535_row_blocks():
    """fp32 blocks of 32 x 32 to a wave: the rows take two launches."""
    torch = torch_mod()
    M, K = 65536 * 32 + 128, 32
    plan = ccl.ccl_plan_typed(M, 128, K, 1, 1, 4096, ccl.CCL_DT_FP32, ccl.CCL_DT_FP32)
    src = torch.randint(-2**31, 2**31 - 1, (K, M), dtype=torch.int32, device="cuda")
    dst = torch.zeros(ccl.ccl_plan_layout(plan, ccl.CCL_A).total_bytes // 4, dtype=torch.int32, device="cuda")
    ccl.ccl_pack(plan, ccl.CCL_A, src, M, 1, dst)
    assert torch.equal(dst[:M * K].view(M, K), src.t())


@pytest.mark.parametrize("rows,ld_extra,off", [(8192, 1, 0), (8320, 0, 1), (8192, 0, 0)])
def test_fp32_above_the_l2s(rows, ld_extra, off):
    """33 to 34 MB of fp32: one element per access off the 16-byte grid."""
    _check(4, rows, 1024, 8 * 129 if off or ld_extra else 8 * 130, 8, 1, "A", False, ld_extra, off, 0, True)


def test_above_the_cache_size():
    """fp32 A of 269 MB in block rows of 1026 elements (4104 bytes)."""
    _check(4, 8192, 1024, 8 * 1026, 8, 1, "A", False, 1, 0, 0, True)
