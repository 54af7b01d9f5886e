// Workgroup -> output-tile map of the GEMM launch, shared by the host plan
// (test hook) and the kernel.
//
// Workgroups are dispatched to the 8 XCDs round-robin (workgroup w runs on
// XCD w mod 8). Chiplet c of G owns XCDs c*8/G .. c*8/G + 8/G - 1 and the
// output partition c (Sec. III-A: each CTA runs on the chiplet owning its
// tile). XCD x of chiplet c takes a contiguous range of that partition's
// tiles, walked in a grouped raster (group_m tile rows at a time) so that
// the tiles resident on one XCD at once share A row panels and B column
// panels in that XCD's L2.
//
// With split-K (splits > 1) every tile is computed as `splits` K ranges by
// separate workgroups of the same XCD: the XCD's range then covers tiles x
// splits virtual tiles, split-major, so that the workgroups resident
// together work on the same K range of neighbouring tiles.
#pragma once

#include <cstdint>

#if defined(__HIPCC__)
#define CCL_HD __host__ __device__ __forceinline__
#else
#define CCL_HD inline
#endif

namespace ccl {

// n / d for 0 <= n < 2^31 by a multiplication: d <= 2^shift, mul =
// ceil(2^(31 + shift) / d), so mul d - 2^(31 + shift) < 2^shift and the
// truncation is exact. A launch's first loads wait for its tile map, and gfx950
// has no integer division: the six of a map were most of the time before them.
struct FastDiv {
  uint32_t mul;
  uint32_t shift;
};

inline FastDiv fast_div(int32_t d) {
  FastDiv f{0, 0};
  while (((int64_t)1 << f.shift) < d) ++f.shift;
  f.mul = (uint32_t)((((uint64_t)1 << (31 + f.shift)) + (uint64_t)d - 1) / (uint64_t)d);
  return f;
}

CCL_HD int32_t operator/(int32_t n, const FastDiv& f) {
  return (int32_t)((((uint64_t)((uint32_t)n << 1) * f.mul) >> 32) >> f.shift);
}

struct TileMap {
  int32_t xcd_per_chip;   // 8 / G
  int32_t grid_c;         // Gc
  int32_t tiles_m;        // kernel tiles per partition, rows
  int32_t tiles_n;        //                              cols
  int32_t tiles_per_xcd;  // ceil(tiles_m * tiles_n * splits / xcd_per_chip)
  int32_t group_m;        // raster group height
  int32_t splits;         // K splits per tile (1: none)
  // divisors of the map: tiles per split, tiles per raster group, the height
  // of a whole group and of the last one
  FastDiv by_tiles, by_group, by_height, by_last;
};

inline TileMap make_tile_map(int32_t xcd_per_chip, int32_t grid_c, int32_t tiles_m, int32_t tiles_n,
                             int32_t tiles_per_xcd, int32_t group_m, int32_t splits) {
  const int32_t last = tiles_m % group_m ? tiles_m % group_m : group_m;
  return TileMap{xcd_per_chip, grid_c, tiles_m, tiles_n, tiles_per_xcd, group_m, splits,
                 fast_div(tiles_m * tiles_n), fast_div(group_m * tiles_n), fast_div(group_m), fast_div(last)};
}

// Returns false when workgroup wg has no tile. Otherwise pr/pc is the
// owning partition, (ti, tj) the tile inside it and split its K range.
// xcd_per_chip and grid_c divide the 8 XCDs; a partition has at most 2^26
// tiles of at most 16 splits, so every count fits in 31 bits.
CCL_HD bool map_tile(const TileMap& m, int64_t wg, int32_t* pr, int32_t* pc, int32_t* ti,
                     int32_t* tj, int32_t* split) {
  const int32_t xcd = (int32_t)(wg & 7);
  const int64_t slot = wg >> 3;
  if (slot >= m.tiles_per_xcd) return false;
  // xcd / xcd_per_chip and chip / grid_c, both powers of two up to 8
  const int32_t xs = (m.xcd_per_chip > 1) + (m.xcd_per_chip > 2) + (m.xcd_per_chip > 4);
  const int32_t cs = (m.grid_c > 1) + (m.grid_c > 2) + (m.grid_c > 4);
  const int32_t chip = xcd >> xs;
  const int32_t sub = xcd & (m.xcd_per_chip - 1);
  const int32_t tiles = m.tiles_m * m.tiles_n;
  const int32_t v = sub * m.tiles_per_xcd + (int32_t)slot;
  if (v >= tiles * m.splits) return false;
  *split = m.splits == 1 ? 0 : v / m.by_tiles;
  const int32_t t = v - *split * tiles;
  const int32_t grp = t / m.by_group;
  const int32_t first = grp * m.group_m;
  const int32_t within = t - first * m.tiles_n;
  const bool whole = m.tiles_m - first >= m.group_m;
  const int32_t gm = whole ? m.group_m : m.tiles_m - first;
  *tj = within / (whole ? m.by_height : m.by_last);
  *ti = first + within - *tj * gm;
  *pr = chip >> cs;
  *pc = chip & (m.grid_c - 1);
  return true;
}

CCL_HD bool map_tile(const TileMap& m, int64_t wg, int32_t* pr, int32_t* pc, int32_t* ti,
                     int32_t* tj) {
  int32_t split;
  return map_tile(m, wg, pr, pc, ti, tj, &split);
}

}  // namespace ccl
