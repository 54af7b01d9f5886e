"""What ccl_gemm itself launches (ccl_debug_launch), against the plan's tile:
the 128x192 and 128x320 tiles' workgroup map against its definition in plain
integers, every tile once and on an XCD of its chiplet; and the kernel form the
dispatch chooses at its edges. No GPU needed."""
import pytest

from oracle import plan as OP
from paper_2606_11718_amd import ccl
from tests.test_host_tile_map import _expected

FP8, BF16, FP32 = ccl.CCL_DT_FP8_E4M3, ccl.CCL_DT_BF16, ccl.CCL_DT_FP32


@pytest.mark.parametrize("wide,G,Gr,tiles_m,tiles_n", [
    (192, 8, 2, 16, 2), (192, 1, 1, 9, 5), (192, 4, 2, 10, 2), (192, 2, 1, 3, 7), (192, 8, 8, 17, 4),
    (320, 8, 1, 15, 2), (320, 1, 1, 11, 3), (320, 4, 1, 8, 5), (320, 8, 4, 19, 2), (320, 2, 2, 1, 9)])
def test_wide_map(wide, G, Gr, tiles_m, tiles_n, monkeypatch):
    monkeypatch.setenv("CCL_GEMM_WIDE", str(wide))
    Gc = G // Gr
    M, N, K = 128 * tiles_m * Gr, wide * 2 * tiles_n * Gc, 512
    tiles_n *= 2                              # partitions hold whole 128-column model tiles
    plan = ccl.ccl_plan(M, N, K, G, Gr, 4096)
    run = ccl.ccl_debug_launch(plan)
    assert (run.kernel, run.tile_rows, run.tile_cols, run.waves) == ("gemm_k64_kernel", 128, wide, 8)
    per_xcd = -(-tiles_m * tiles_n // (8 // G))
    assert run.workgroups == 8 * per_xcd
    seen = set()
    for wg in range(run.workgroups + 8):
        xcd, ti, tj = ccl.ccl_debug_launch_tile_of_wg(plan, wg)
        assert (xcd, (ti, tj)) == (wg % 8, _expected(wg, G, Gr, tiles_m, tiles_n, min(8, tiles_m))), wg
        if ti >= 0:
            assert (ti, tj) not in seen
            seen.add((ti, tj))
            owners = {OP.owner(ti, c // 128, M, N, Gr, Gc) for c in (tj * wide, (tj + 1) * wide - 1)}
            assert len(owners) == 1 and xcd in OP.xcds_of_chiplet(owners.pop(), G)
    assert len(seen) == G * tiles_m * tiles_n


@pytest.mark.parametrize("M,N,K,G,Gr,cols", [
    (4096, 1536, 2048, 8, 2, 192), (256, 16896, 1280, 8, 2, 192), (2048, 4608, 1024, 8, 2, 192),
    (3840, 3072, 512, 8, 2, 192), (7680, 768, 2048, 8, 4, 192),
    (4096, 3072, 2048, 8, 2, 256), (7680, 1536, 512, 4, 2, 256), (2048, 6144, 4096, 4, 2, 256),
    (2048, 12288, 2048, 8, 2, 128),
    (1920, 5120, 1792, 8, 1, 320), (2560, 7680, 512, 8, 2, 320), (15360, 1280, 1024, 8, 8, 320),
    (7680, 5120, 4096, 8, 4, 256), (12288, 3200, 1024, 8, 8, 128), (1024, 5120, 4096, 8, 2, 128)])
def test_wide_tiles_where_they_measured_faster(M, N, K, G, Gr, cols):
    assert ccl.ccl_debug_launch(ccl.ccl_plan(M, N, K, G, Gr, 4096)).tile_cols == cols


@pytest.mark.parametrize("group", [1, 3, 4, 8, 16])
def test_raster_override_reaches_wide_tiles(group, monkeypatch):
    """CCL_GEMM_GROUP_M sets the raster height of every launch."""
    monkeypatch.setenv("CCL_GEMM_GROUP_M", str(group))
    plan = ccl.ccl_plan(4096, 1536, 2048, 8, 2, 4096)
    assert ccl.ccl_debug_launch(plan).tile_cols == 192
    for wg in range(256):
        assert ccl.ccl_debug_launch_tile_of_wg(plan, wg)[1:] == _expected(wg, 8, 2, 16, 2, group), wg


def test_chosen_wide_tiles_and_the_plan_tile():
    """The plan's tile stays what split-K uses; the launch hook says what runs."""
    plan = ccl.ccl_plan(4096, 1536, 2048, 8, 2, 4096)
    assert ccl.ccl_debug_gemm_config(plan)[:2] == (256, 128)
    run = ccl.ccl_debug_launch(plan)
    assert (run.tile_rows, run.tile_cols, run.workgroups, run.k_ranges) == (128, 192, 256, 1)
    split = ccl.ccl_debug_launch(plan, 2)
    assert (split.kernel, split.tile_rows, split.tile_cols, split.k_ranges) == ("gemm_k64_kernel", 256, 128, 2)
    assert ccl.ccl_debug_launch(plan, 1, 2).tile_cols == 192           # row-major, XCD-aware map
    assert ccl.ccl_debug_launch(plan, 1, 1).tile_cols == 128           # row-major, native order


@pytest.mark.parametrize("shape,env,kernel,ragged", [
    ((1024, 1024, 1024, 8, 2, BF16), {"CCL_GEMM_TILE": "128x128"}, "gemm_k64_kernel", False),
    ((1024, 1024, 1024, 8, 2, BF16), {"CCL_GEMM_TILE": "128x128", "CCL_GEMM_STAGE_K": "32"}, "gemm_kernel", False),
    ((1024, 1024, 1024, 8, 2, BF16), {"CCL_GEMM_TILE": "128x128", "CCL_GEMM_WAVES": "4"}, "gemm_kernel", False),
    ((256, 256, 32, 1, 1, BF16), {}, "gemm_kernel", False),            # K blocks of one 32-K step
    ((256, 256, 96, 1, 1, BF16), {"CCL_GEMM_TILE": "128x128"}, "gemm_k64_kernel", True),
    ((8192, 28672, 8192, 8, 2, BF16), {}, "gemm_a2_kernel", False),
    ((8192, 28672, 8192, 8, 2, FP8), {}, "gemm_fp8p_kernel", False),
    ((8192, 28672, 8192, 8, 2, FP8), {"CCL_GEMM_FP8_PIPE": "0"}, "gemm_fp8x_kernel", False),
    ((4096, 1536, 2048, 8, 2, FP8), {}, "gemm_fp8s_kernel", False),
    ((4096, 1536, 2112 * 4, 8, 2, FP8), {"CCL_GEMM_TILE": "256x128"}, "gemm_fp8_kernel", False),  # 64 mod 128
])
def test_form(shape, env, kernel, ragged, monkeypatch):
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    M, N, K, G, Gr, ab = shape
    run = ccl.ccl_debug_launch(ccl.ccl_plan_typed(M, N, K, G, Gr, 4096, ab, BF16))
    assert (run.kernel, run.ragged) == (kernel, ragged)


@pytest.mark.parametrize("M,N,K,G,Gr,stream", [
    (128, 28672, 8192, 8, 1, True), (128, 28672, 8192, 1, 1, True),
    (128, 16384, 8192, 8, 1, False),          # 256 MiB: stays in the Infinity Cache
    (128, 16384, 8448, 8, 1, True),
    (256, 28672, 8192, 8, 1, False),          # two tile rows
    (256, 28672, 8192, 8, 2, False), (512, 28672, 8192, 8, 4, False), (1024, 28672, 8192, 8, 8, False),
    (256, 24576, 8192, 8, 2, False), (512, 20480, 8192, 8, 4, False)])
def test_b_streams_where_one_workgroup_reads_it(M, N, K, G, Gr, stream, monkeypatch):
    if M == 256 and Gr == 1:
        monkeypatch.setenv("CCL_GEMM_TILE", "128x256")
    assert ccl.ccl_debug_launch(ccl.ccl_plan(M, N, K, G, Gr, 4096)).stream_b == stream


@pytest.mark.parametrize("M,N,c,nt", [
    (2048, 4096, FP32, False), (8192, 4096, FP32, False), (8192, 8192 - 128 * 8, FP32, False),
    (8192, 8192, FP32, True), (8192, 28672, FP32, True),
    (8192, 12288, BF16, False), (8192, 16384, BF16, True), (8192, 28672, BF16, True)])
@pytest.mark.parametrize("ab", [BF16, FP8])
def test_c_leaves_the_cache_only_above_its_size(M, N, c, nt, ab):
    """An fp32 C counts alone, a bf16 C together with the operands (K 1024)."""
    plan = ccl.ccl_plan_typed(M, N, 1024, 8, 2, 4096, ab, c)
    assert ccl.ccl_debug_launch(plan).c_nt == nt
    assert ccl.ccl_debug_launch(plan, operands=2).c_nt == nt
    assert ccl.ccl_debug_launch(plan, operands=1).c_nt == (nt or c == BF16)      # row-major, native order


@pytest.mark.parametrize("M,N,K,G,Gr,splits,far,stream", [
    (128, 131072, 8192, 1, 1, 1, True, True),        # B of 2 GiB in one block: a vocabulary projection in decode
    (128, 131072, 8192, 1, 1, 4, True, True),
    (128, 130048, 8192, 1, 1, 1, False, True),
    (128, 131072, 8192, 8, 1, 1, False, True),       # in 8 column blocks, one to a tile
    (256, 262144, 8192, 8, 2, 1, True, False),       # in 2 x 4 blocks: a tile spans 5/8 of 4 GiB
    (131072, 1024, 9728, 8, 1, 1, True, False),      # A in 8 K blocks
    (131072, 128, 9728, 1, 1, 1, False, False),      # one K block of A: a tile spans 256 rows only
])
def test_64k_stages_above_two_gib(M, N, K, G, Gr, splits, far, stream):
    run = ccl.ccl_debug_launch(ccl.ccl_plan(M, N, K, G, Gr, 4096), splits)
    assert (run.kernel, run.ragged, run.far, run.stream_b) == ("gemm_k64_kernel", False, far, stream)


def test_ragged_blocks_above_two_gib_keep_the_32k_kernel():
    run = ccl.ccl_debug_launch(ccl.ccl_plan(128, 131072, 8224, 1, 1, 4096))      # 257 steps
    assert (run.kernel, run.far) == ("gemm_kernel", False)


@pytest.mark.parametrize("tile,M,N,K,G,Gr,ragged64", [
    ("128x256", 256, 8192, 2304, 8, 1, False), ("128x256", 640, 12288, 4352, 8, 1, False),
    ("128x256", 384, 22528, 8448, 8, 1, True),       # 387 MB
    ("128x256", 2048, 1024, 8224, 1, 1, False),
    ("256x128", 512, 4096, 768, 8, 1, False), ("256x128", 1024, 4096, 1280, 8, 1, False),
    ("256x128", 1024, 4096, 1792, 8, 1, True), ("256x128", 1536, 1408, 2080, 1, 1, True),
    ("128x128", 512, 8192, 768, 8, 1, True),         # 32 tiles per XCD
    ("128x128", 384, 11264, 768, 8, 1, False),       # 33
])
def test_ragged_64k_stages_where_they_pay(tile, M, N, K, G, Gr, ragged64, monkeypatch):
    monkeypatch.setenv("CCL_GEMM_TILE", tile)
    run = ccl.ccl_debug_launch(ccl.ccl_plan(M, N, K, G, Gr, 4096))
    assert (run.kernel, run.ragged) == (("gemm_k64_kernel", True) if ragged64 else ("gemm_kernel", False))
    monkeypatch.setenv("CCL_GEMM_STAGE_K", "64")
    run = ccl.ccl_debug_launch(ccl.ccl_plan(M, N, K, G, Gr, 4096))
    assert (run.kernel, run.ragged) == ("gemm_k64_kernel", True)


@pytest.mark.parametrize("N,K,splits,kernel", [
    (3072, 2048, 2, "gemm_fp8s_kernel"), (3072, 2048, 4, "gemm_fp8_kernel"),        # 18 and 36 workgroups per XCD
    (5120, 2048, 2, "gemm_fp8s_kernel"), (5120, 4096, 4, "gemm_fp8_kernel"),        # 30 and 60
    (11264, 2048, 1, "gemm_fp8s_kernel")])
def test_fp8_split_ranges_share_cus(N, K, splits, kernel):
    plan = ccl.ccl_plan_typed(384, N, K, 8, 1, 4096, FP8, BF16)
    run = ccl.ccl_debug_launch(plan, splits)
    assert (run.tile_rows, run.tile_cols, run.kernel, run.waves) == (128, 128, kernel, 4 if kernel == "gemm_fp8_kernel" else 8)


@pytest.mark.parametrize("N,K,c,reads_c,kernel", [
    (9216, 1024, FP32, 0, "gemm_fp8_kernel"), (9216, 1024, FP32, 1, "gemm_fp8s_kernel"),     # 45 tiles per XCD
    (9216, 2048, FP32, 0, "gemm_fp8_kernel"), (9216, 3072, FP32, 0, "gemm_fp8s_kernel"),
    (9216, 1024, BF16, 0, "gemm_fp8s_kernel"), (5120, 1024, FP32, 0, "gemm_fp8s_kernel")])   # 25 tiles
def test_fp8_tiles_with_an_fp32_c_share_cus(N, K, c, reads_c, kernel):
    run = ccl.ccl_debug_launch(ccl.ccl_plan_typed(640, N, K, 8, 1, 4096, FP8, c), reads_c=reads_c)
    assert (run.tile_rows, run.tile_cols, run.kernel) == (128, 128, kernel)


def test_odd_k_ranges_of_whole_blocks_keep_32k_stages():
    plan = ccl.ccl_plan(2048, 256, 6016, 4, 2, 4096)
    assert ccl.ccl_debug_launch(plan, 3).kernel == "gemm_kernel"           # 63 steps
    run = ccl.ccl_debug_launch(plan, 2)                                    # 94
    assert (run.kernel, run.ragged) == ("gemm_k64_kernel", False)


def test_arguments():
    plan = ccl.ccl_plan(1024, 1024, 1024, 8, 2, 4096)
    for splits, operands in ((0, 0), (17, 0), (1, 3), (1, -1), (2, 1)):
        with pytest.raises(ccl.CCLError, match="CCL_ERR_INVALID_ARG"):
            ccl.ccl_debug_launch(plan, splits, operands)
    for operands, reads_c in ((0, 2), (0, -1), (1, 1)):
        with pytest.raises(ccl.CCLError, match="CCL_ERR_INVALID_ARG"):
            ccl.ccl_debug_launch(plan, 1, operands, reads_c)
    with pytest.raises(ccl.CCLError, match="CCL_ERR_UNSUPPORTED"):
        ccl.ccl_debug_launch(ccl.ccl_plan_typed(384, 768, 384, 3, 1, 4096, BF16, BF16))
