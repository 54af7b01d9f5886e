"""The workgroup -> tile map against its definition in plain integers (the map
itself divides by multiplication), over raster groups that do and do not divide
the tile rows, every grid, and counts up to the largest plans. No GPU needed."""
import pytest

from paper_2606_11718_amd import ccl


def _expected(wg, G, Gr, tiles_m, tiles_n, group):
    xpc, Gc = 8 // G, G // Gr
    per_xcd = -(-tiles_m * tiles_n // xpc)
    chip, sub = (wg % 8) // xpc, (wg % 8) % xpc
    t = sub * per_xcd + wg // 8
    if wg // 8 >= per_xcd or t >= tiles_m * tiles_n:
        return -1, -1
    first = t // (group * tiles_n) * group
    height = min(group, tiles_m - first)
    within = t - first * tiles_n
    return chip // Gc * tiles_m + first + within % height, chip % Gc * tiles_n + within // height


@pytest.mark.parametrize("group", [1, 3, 4, 8])
@pytest.mark.parametrize("G,Gr,tiles_m,tiles_n", [
    (1, 1, 1, 1), (1, 1, 7, 5), (2, 1, 9, 11), (4, 2, 13, 3), (8, 1, 1, 31), (8, 2, 17, 6), (8, 4, 5, 29),
    (8, 8, 33, 1), (8, 2, 1023, 1021)])
def test_map_is_its_definition(G, Gr, tiles_m, tiles_n, group, monkeypatch):
    monkeypatch.setenv("CCL_GEMM_TILE", "128x128")
    monkeypatch.setenv("CCL_GEMM_GROUP_M", str(group))
    Gc = G // Gr
    plan = ccl.ccl_plan(128 * tiles_m * Gr, 128 * tiles_n * Gc, 256, G, Gr, 4096)
    wgs = ccl.ccl_debug_gemm_config(plan)[2]
    group = min(group, tiles_m)
    step = 1 if wgs < 20000 else 9973
    for wg in list(range(0, wgs, step)) + [wgs - 1]:
        xcd, ti, tj = ccl.ccl_debug_tile_of_wg(plan, wg)
        assert (xcd, (ti, tj)) == (wg % 8, _expected(wg, G, Gr, tiles_m, tiles_n, group)), wg
