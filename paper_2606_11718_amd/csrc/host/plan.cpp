// Host-side plan of a CCL GEMM (see plan.hpp).
//
// Remote-byte model (Sec. IV-A "Metrics"; no cache): every 128x128 output
// tile runs on its owner chiplet, reads its whole A row panel and B column
// panel and writes its C tile; an element access is remote when the page
// holding the element sits on another chiplet. The model here walks, for
// each panel, the byte intervals the panel occupies in the stored tensor
// and splits every interval at page boundaries, so the per-chiplet counts
// come from interval lengths rather than from element enumeration.
#include "plan.hpp"

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

namespace ccl {

namespace {

bool is_pow2(int64_t x) { return x > 0 && (x & (x - 1)) == 0; }

Layout make_layout(int64_t rows, int64_t cols, int Gr, int Gc, int64_t page, int e) {
  Layout l;
  l.elem_bytes = e;
  l.rows = rows;
  l.cols = cols;
  l.grid_r = Gr;
  l.grid_c = Gc;
  l.block_rows = rows / Gr;
  l.block_cols = cols / Gc;
  l.strip_bytes = l.block_rows * l.block_cols * e;
  l.strip_stride_bytes = (l.strip_bytes + page - 1) / page * page;
  l.total_bytes = l.strip_stride_bytes * Gr * Gc;
  return l;
}

// Extra bytes of the shared operands that their non-owning sharers need,
// scaled by G to stay an integer: e_A*M*K*(Gc-1)*Gr + e_B*K*N*(Gr-1)*Gc.
unsigned __int128 replicated_times_g(int64_t M, int64_t N, int64_t K, int Gr, int Gc, int ea, int eb) {
  unsigned __int128 a = (unsigned __int128)M * K * (Gc - 1) * Gr * ea;
  unsigned __int128 b = (unsigned __int128)K * N * (Gr - 1) * Gc * eb;
  return a + b;
}

// Panels (distinct tile rows plus distinct tile columns) that the waves of
// 32 co-resident tiles touch, summed over the XCDs of one chiplet, when each
// XCD walks its range of the partition's tiles in groups of gm tile rows,
// each group column by column (the order of map_tile in tile_map.hpp).
int64_t panels_touched(const GemmConfig& g, int gm) {
  const int64_t tiles = g.tiles_m * g.tiles_n;
  const int64_t h0 = std::min<int64_t>(gm, g.tiles_m);
  const int64_t per_group = h0 * g.tiles_n;
  int64_t total = 0;
  std::vector<char> row_seen(g.tiles_m), col_seen(g.tiles_n);
  for (int64_t sub = 0; sub < g.xcd_per_chiplet; ++sub) {
    for (int64_t w0 = 0; w0 < g.tiles_per_xcd; w0 += 32) {
      std::fill(row_seen.begin(), row_seen.end(), 0);
      std::fill(col_seen.begin(), col_seen.end(), 0);
      for (int64_t slot = w0; slot < std::min<int64_t>(w0 + 32, g.tiles_per_xcd); ++slot) {
        const int64_t t = sub * g.tiles_per_xcd + slot;
        if (t >= tiles) break;
        const int64_t first = (t / per_group) * h0;
        const int64_t h = std::min<int64_t>(h0, g.tiles_m - first);
        const int64_t w = t - (t / per_group) * per_group;
        const int64_t ti = first + w % h, tj = w / h;
        total += (row_seen[ti] ? 0 : 1) + (col_seen[tj] ? 0 : 1);
        row_seen[ti] = col_seen[tj] = 1;
      }
    }
  }
  return total;
}

void choose_gemm_config(Plan* p) {
  GemmConfig& g = p->gemm;
  g = GemmConfig();
  const int64_t pr = p->part_rows(), pc = p->part_cols();
  if (kNumXcd % p->G != 0) {
    g.why_unsupported = "chiplets must divide the 8 XCDs";
    return;
  }
  if (p->ab_type == DT_FP32) {
    g.why_unsupported = "the GEMM kernels take bf16 or fp8 A and B (fp32 plans serve layouts and traffic models)";
    return;
  }
  const int64_t bk = p->ab_type == DT_FP8_E4M3 ? kGemmBK8 : kGemmBK;
  if ((p->K / p->Gc) % bk != 0 || (p->K / p->Gr) % bk != 0) {
    g.why_unsupported = p->ab_type == DT_FP8_E4M3
                            ? "fp8: K / grid_cols and K / grid_rows must be multiples of 64"
                            : "K / grid_cols and K / grid_rows must be multiples of 32";
    return;
  }
  g.xcd_per_chiplet = kNumXcd / p->G;
  // Candidate kernel tiles, largest first; estimated time = waves of 32
  // workgroups per XCD times the tile's work over a per-tile efficiency.
  struct Cand { int tm, tn; double eff; };
  const Cand cands[] = {{256, 256, 1.0}, {256, 128, 0.85}, {128, 256, 0.85}, {128, 128, 0.7}};
  double best = 0;
  int btm = 0, btn = 0;
  const char* forced = std::getenv("CCL_GEMM_TILE");
  int ftm = 0, ftn = 0;
  if (forced && std::sscanf(forced, "%dx%d", &ftm, &ftn) != 2) ftm = ftn = 0;
  for (const Cand& c : cands) {
    if (pr % c.tm || pc % c.tn) continue;
    if (ftm && (c.tm != ftm || c.tn != ftn)) continue;
    int64_t tiles = (pr / c.tm) * (pc / c.tn);
    int64_t per_xcd = (tiles + g.xcd_per_chiplet - 1) / g.xcd_per_chiplet;
    int64_t waves = (per_xcd + 31) / 32;
    double t = (double)waves * c.tm * c.tn / c.eff;
    if (btm == 0 || t < best) {
      best = t;
      btm = c.tm;
      btn = c.tn;
    }
  }
  if (btm == 0) {
    g.why_unsupported = "no kernel tile fits the partitions (or CCL_GEMM_TILE does not)";
    return;
  }
  g.tile_m = btm;
  g.tile_n = btn;
  g.tiles_m = pr / btm;
  g.tiles_n = pc / btn;
  g.tiles_per_xcd = (g.tiles_m * g.tiles_n + g.xcd_per_chiplet - 1) / g.xcd_per_chiplet;
  g.workgroups = g.tiles_per_xcd * kNumXcd;
  // Raster group height. An XCD runs 32 tiles at once (one workgroup per CU);
  // 4 tile rows x 8 tile columns make them share 12 A row panels and B
  // column panels, which the XCD's L2 serves while they step through K
  // together. Where a group is not a whole number of such waves, some waves
  // straddle two groups and touch more panels. So the height is the one of
  // 4 and 8 whose waves touch the fewest panels in total (4 on a tie: on
  // 8192x8192x28672 both give 12 per wave and 4 measured 1.5 % faster).
  // Measured on 8192x28672x8192 (28 tile columns, 8 rows chosen): 9 % less
  // L2-miss traffic than 4 rows, 1 % faster.
  int gm = panels_touched(g, 8) < panels_touched(g, 4) ? 8 : 4;
  // Wider tiles (below) take 8 rows: 32 resident tiles then cover 1024 x 768 or
  // 1024 x 1280 of C. 4 rows measured 0-6 % slower on six 192-wide and nine
  // 320-wide shapes (7680x3840x512 45.7 -> 48.2 us, 1536x12800x2048 74.3 -> 77.4),
  // 16 rows within 2 % either way.
  g.wide_group_m = 8;
  if (const char* e = std::getenv("CCL_GEMM_GROUP_M")) gm = g.wide_group_m = std::max(1, std::atoi(e));
  g.group_m = (int)std::min<int64_t>(gm, g.tiles_m);
  // Waves per workgroup: 8 (two per SIMD) for every bf16 tile, for fp8
  // 256x256 tiles and for the other fp8 tiles where both K blocks are
  // multiples of 128 (gemm_fp8s_kernel's stage), 4 for fp8 tiles below
  // 256x256 otherwise. On the Qwen3 shapes the 8-wave forms of the bf16
  // 256x128 and 128x128 tiles measured 0-10 % faster than 4.
  // CCL_GEMM_WAVES=4 selects the 4-wave form.
  const bool eight_ok = (btm == 256 && btn == 256) || p->ab_type == DT_BF16 ||
                        ((p->K / p->Gc) % 128 == 0 && (p->K / p->Gr) % 128 == 0);
  g.waves = eight_ok ? 8 : 4;
  if (const char* e = std::getenv("CCL_GEMM_WAVES"))
    g.waves = (std::atoi(e) == 8 && eight_ok) ? 8 : 4;
  // LDS stage depth in K (bf16). A stage of 32 K holds 64-byte A rows, half
  // a 128-byte line, and a CU streams such half lines from L2 at 36-47
  // B/clk when most CUs load, against 57-64 B/clk for whole lines
  // (direct-to-LDS loads of L2-resident data). The tiles below 256x256 need
  // 48-64 B/clk per CU at the matrix cores' rate, so they take 64-K stages
  // (whole-line A rows). 256x256 keeps 32: two 64-K stages would leave one
  // step of load lookahead.
  // CCL_GEMM_STAGE_K=32 selects the 32-K stages everywhere, 64 the 64-K ones
  // wherever they exist (gemm_form has the rules for ragged K blocks).
  g.stage_k = (p->ab_type == DT_BF16 && g.waves == 8 && !(btm == 256 && btn == 256)) ? 64 : 32;
  const char* stage_env = std::getenv("CCL_GEMM_STAGE_K");
  const bool stage32 = stage_env && std::atoi(stage_env) == 32;
  g.stage_64 = stage_env && std::atoi(stage_env) == 64;
  if (stage32) g.stage_k = 32;
  // CCL_GEMM_FAR=1 takes the form for operands of 2 GiB and more at any size.
  if (const char* e = std::getenv("CCL_GEMM_FAR")) g.far = std::atoi(e) == 1;
  // B streams past the L2 where each of its lines is read by one workgroup
  // only (one tile row per partition, one partition row), and it is above the
  // Infinity Cache size (non-temporal lines do not stay there either). Us per
  // launch, not streamed -> streamed: 128x28672x8192 on 1x8 104.4 -> 98.2, on
  // one partition 103.1 -> 96.5. With two, four and eight partition rows the
  // Infinity Cache serves all reads of B but one, and streaming loses:
  // 256x28672x8192 on 2x4 144.6 -> 161.6, 512x28672x8192 on 4x2 282.5 ->
  // 320.5, 1024x28672x8192 on 8x1 571.7 -> 660.6. Below that size a weight
  // that is in the cache must be read from there: the 256x16896x1280 pass
  // (43 MB, pack, GEMM and unpack) took 42.0 us streamed, 37.1 not. Where tile
  // rows share B it is 20-50 % slower. CCL_GEMM_STREAM_B=0|1 overrides the
  // size and partition rules.
  g.stream_b = p->ab_type == DT_BF16 && g.tiles_m == 1;
  if (const char* e = std::getenv("CCL_GEMM_STREAM_B"))
    g.stream_b = g.stream_b && std::atoi(e) != 0;
  else
    g.stream_b = g.stream_b && p->Gr == 1 && p->K * p->N * 2 > kInfinityCacheBytes;
  // 256x256 keeps 32-K steps for B and the MFMA schedule but stages A in
  // 64-K pairs of steps: whole 128-byte lines per A load, and loads four
  // steps ahead in a ring of three pair buffers. Same box, alternating:
  // 8192x28672x8192 1416-1423 -> 1484-1492 TFLOP/s, 8192x8192x28672
  // 1433-1437 -> 1504-1508, at the same 1400 W. Needs A's K blocks in
  // whole pairs. CCL_GEMM_A_PAIRS=0 selects the 32-K A stages.
  g.a_pairs = p->ab_type == DT_BF16 && g.waves == 8 && btm == 256 && btn == 256 &&
              (p->K / p->Gc) % 64 == 0;
  if (const char* e = std::getenv("CCL_GEMM_A_PAIRS"))
    if (std::atoi(e) == 0) g.a_pairs = false;
  // fp8 256x256 (16x16x128 kernel): three A and two B stage buffers, two
  // barriers per step, and the next step's fragments read behind the last
  // rows of MFMAs (gemm_fp8p_kernel). CCL_GEMM_FP8_PIPE=0 selects the
  // two-stage kernel that reads them after each step's barrier.
  g.fp8_pipe = p->ab_type == DT_FP8_E4M3 && g.waves == 8 && btm == 256 && btn == 256;
  if (const char* e = std::getenv("CCL_GEMM_FP8_PIPE"))
    if (std::atoi(e) == 0) g.fp8_pipe = false;
  // 128x192 and 128x320 tiles for unsplit bf16 launches where their waves of
  // 32 per XCD cost less than the tile above (same estimate). They fill
  // partitions whose 128- or 256-wide tiles leave CUs idle: 4096x1536x2048
  // (2048x384 per XCD, 24 tiles of 256x128, now 32) 33.9 -> 31.9 us a launch,
  // 256x16896x1280 (33 tiles of 128x128, now 22) 27.6 -> 17.9; 1920x5120x1792
  // (75 tiles of 128x128, now 30 of 128x320) 52.5 -> 42.4, 2048x5120x2048 54 ->
  // 44.5, 4096x2560x4096 90 -> 73.
  // The estimate orders the measured launches by their gain, so each width's
  // efficiency lies between the ones that gain and the ones that do not:
  //  * 192 (four stages): plans that need 0.700 gain 8-11 % (five shapes), those
  //    that need 0.750 0-4 %, or lose up to 4 % (24 tiles of 256x256:
  //    4096x3072x2048 52.6 -> 54.8, 7680x1536x512 19.0 -> 19.4; five shapes).
  //  * 320 (two stages): at 0.708 8-13 % (five shapes), at 0.781 and 0.797 3 and
  //    7 % (one shape each), at 0.850 1 % to -4 % (four shapes).
  // The kernel has 64-K stages, K blocks of at least one, and 31-bit extents.
  // CCL_GEMM_WIDE=0|192|320 forbids them / takes that one wherever it exists.
  {
    const int64_t lim = ((int64_t)1 << 31) - 4096;
    const Layout &la = p->lay[OP_A], &lb = p->lay[OP_B];
    const bool exists = p->ab_type == DT_BF16 && pr % 128 == 0 && g.waves == 8 &&
                        (g.stage_k == 64 || (btm == 256 && btn == 256 && !stage32)) && !forced &&
                        p->K / p->Gc >= 64 && p->K / p->Gr >= 64 &&
                        la.strip_stride_bytes * p->Gc + 512 * p->K < lim && lb.total_bytes + 512 < lim;
    const char* e = std::getenv("CCL_GEMM_WIDE");
    const int forced_n = e ? std::atoi(e) : -1;
    double t = best;
    for (int n : {192, 320}) {
      if (!exists || pc % n || (e && n != forced_n)) continue;
      const int64_t tiles = (pr / 128) * (pc / n);
      const int64_t waves = ((tiles + g.xcd_per_chiplet - 1) / g.xcd_per_chiplet + 31) / 32;
      const double tn = (double)waves * 128 * n / (n == 192 ? 0.725 : 0.75);
      if (e || tn < t) {
        t = tn;
        g.wide_n = n;
      }
    }
  }
  if (g.workgroups > 0x7fffffff) {
    g.why_unsupported = "launch too large";
    return;
  }
  g.supported = true;
}

// Per-chiplet element counts of rectangles of one stored operand.
struct Placed {
  int64_t R, Cc;      // logical shape
  bool trans;         // stored as the transpose (Cc x R row-major)
  Placement pl;
  const Layout* lay;
  int G;
  int64_t page;
  int64_t n_pages;    // pages of the stored row-major tensor
  int64_t e;          // element bytes

  int chip_of_page(int64_t pg) const {
    if (pl == PLACE_RR) return (int)(pg % G);
    return (int)((pg * (int64_t)G) / n_pages);   // coarse: G contiguous chunks
  }

  // Bytes [s0, s1) of the stored tensor, split at page boundaries.
  void add_interval(int64_t s0, int64_t s1, uint64_t* h) const {
    int64_t pg = s0 / page;
    while (s0 < s1) {
      int64_t end = std::min((pg + 1) * page, s1);
      h[chip_of_page(pg)] += (uint64_t)((end - s0) / e);
      s0 = end;
      ++pg;
    }
  }

  // Add per-chiplet counts of logical rectangle [r0,r1) x [c0,c1) to h.
  void count(int64_t r0, int64_t r1, int64_t c0, int64_t c1, uint64_t* h) const {
    if (pl == PLACE_CCL) {
      const int64_t hr = lay->block_rows, wc = lay->block_cols;
      for (int64_t br = r0 / hr; br * hr < r1; ++br) {
        int64_t ro = std::min(r1, (br + 1) * hr) - std::max(r0, br * hr);
        for (int64_t bc = c0 / wc; bc * wc < c1; ++bc) {
          int64_t co = std::min(c1, (bc + 1) * wc) - std::max(c0, bc * wc);
          h[br * lay->grid_c + bc] += (uint64_t)(ro * co);
        }
      }
      return;
    }
    if (!trans) {
      for (int64_t r = r0; r < r1; ++r)
        add_interval((r * Cc + c0) * e, (r * Cc + c1) * e, h);
    } else {
      for (int64_t c = c0; c < c1; ++c)
        add_interval((c * R + r0) * e, (c * R + r1) * e, h);
    }
  }
};

}  // namespace

bool grid_aligned(int64_t M, int64_t N, int64_t K, int G, int Gr) {
  if (Gr <= 0 || G % Gr != 0) return false;
  int Gc = G / Gr;
  return M % ((int64_t)Gr * kModelTile) == 0 && N % ((int64_t)Gc * kModelTile) == 0 &&
         K % Gr == 0 && K % Gc == 0;
}

uint64_t floor_bytes(int64_t M, int64_t N, int64_t K, int Gr, int Gc, int ea, int eb) {
  // A: each element read by Gc chiplets, N/(Gc*128) times each, one of them local.
  unsigned __int128 a = (unsigned __int128)M * K * (N / ((int64_t)Gc * kModelTile)) * (Gc - 1) * ea;
  unsigned __int128 b = (unsigned __int128)K * N * (M / ((int64_t)Gr * kModelTile)) * (Gr - 1) * eb;
  return (uint64_t)(a + b);
}

Status make_plan(int64_t M, int64_t N, int64_t K, int chiplets, int grid_rows, int64_t page,
                 DType ab, DType c, Plan* out, std::string* err) {
  if (!out) {
    *err = "plan output pointer is NULL";
    return Status::INVALID_ARG;
  }
  if (M <= 0 || N <= 0 || K <= 0) {
    *err = "M, N and K must be positive";
    return Status::INVALID_ARG;
  }
  const int64_t lim = (int64_t)1 << 31;
  if (M >= lim || N >= lim || K >= lim ||
      (unsigned __int128)M * N * K >= ((unsigned __int128)1 << 62) ||
      (unsigned __int128)M * K >= ((unsigned __int128)1 << 40) ||
      (unsigned __int128)K * N >= ((unsigned __int128)1 << 40) ||
      (unsigned __int128)M * N >= ((unsigned __int128)1 << 40)) {
    *err = "problem size overflows the 64-bit byte counts";
    return Status::INVALID_ARG;
  }
  if (chiplets < 1 || chiplets > kMaxChiplets) {
    *err = "chiplets must be in 1..64";
    return Status::INVALID_ARG;
  }
  if (!is_pow2(page) || page < 128 || page > ((int64_t)1 << 40)) {
    *err = "page_bytes must be a power of two in [128, 2^40]";
    return Status::INVALID_ARG;
  }
  if ((ab != DT_BF16 && ab != DT_FP8_E4M3 && ab != DT_FP32) || (c != DT_BF16 && c != DT_FP32)) {
    *err = "A and B must be bf16, fp8 E4M3 or fp32, C bf16 or fp32";
    return Status::INVALID_ARG;
  }
  const int ea = dtype_bytes(ab), ec = dtype_bytes(c);
  if (grid_rows < 0 || (grid_rows > 0 && chiplets % grid_rows != 0)) {
    *err = "grid_rows must be 0 (automatic) or divide chiplets";
    return Status::INVALID_ARG;
  }
  int Gr = grid_rows;
  if (Gr == 0) {
    // Fewest CCL remote bytes (= floor), then fewest replicated shared
    // bytes, then the smaller grid_rows.
    bool found = false;
    uint64_t best_floor = 0;
    unsigned __int128 best_rep = 0;
    for (int r = 1; r <= chiplets; ++r) {
      if (!grid_aligned(M, N, K, chiplets, r)) continue;
      uint64_t f = floor_bytes(M, N, K, r, chiplets / r, ea, ea);
      unsigned __int128 rep = replicated_times_g(M, N, K, r, chiplets / r, ea, ea);
      if (!found || f < best_floor || (f == best_floor && rep < best_rep)) {
        found = true;
        best_floor = f;
        best_rep = rep;
        Gr = r;
      }
    }
    if (!found) {
      *err = "no grid gives 128-aligned partitions";
      return Status::UNALIGNED;
    }
  } else if (!grid_aligned(M, N, K, chiplets, Gr)) {
    *err = "partitions must be multiples of 128x128 tiles and K divisible by both grid sides";
    return Status::UNALIGNED;
  }
  Plan p;
  p.M = M;
  p.N = N;
  p.K = K;
  p.G = chiplets;
  p.Gr = Gr;
  p.Gc = chiplets / Gr;
  p.page = page;
  p.ab_type = ab;
  p.c_type = c;
  p.lay[OP_A] = make_layout(M, K, p.Gr, p.Gc, page, ea);
  p.lay[OP_B] = make_layout(K, N, p.Gr, p.Gc, page, ea);
  p.lay[OP_C] = make_layout(M, N, p.Gr, p.Gc, page, ec);
  choose_gemm_config(&p);
  *out = p;
  return Status::OK;
}

Traffic remote_bytes(const Plan& p, Placement pl, int flags) {
  const int trans_mask = flags & 3;
  const uint64_t c_times = (flags & kTrafficCRead) ? 2 : 1;   // beta != 0: C read, then written
  Traffic t;
  t.chiplets = p.G;
  const int G = p.G;
  const int64_t T = kModelTile;
  const int64_t TM = p.M / T, TN = p.N / T;
  const int64_t tm_per_part = p.part_rows() / T, tn_per_part = p.part_cols() / T;
  const int64_t shapes[3][2] = {{p.M, p.K}, {p.K, p.N}, {p.M, p.N}};
  Placed ops[3];
  for (int o = 0; o < 3; ++o) {
    const int64_t e = p.lay[o].elem_bytes;
    int64_t bytes = shapes[o][0] * shapes[o][1] * e;
    ops[o] = Placed{shapes[o][0], shapes[o][1], o < 2 && ((trans_mask >> o) & 1), pl,
                    &p.lay[o],   G,            p.page, (bytes + p.page - 1) / p.page, e};
    t.footprint[o] = pl == PLACE_CCL ? (uint64_t)p.lay[o].total_bytes : (uint64_t)bytes;
  }
  std::vector<uint64_t> h(G);
  const uint64_t ea = p.lay[OP_A].elem_bytes, eb = p.lay[OP_B].elem_bytes, ec = p.lay[OP_C].elem_bytes;

  // A: row panel ti is read by the TN tiles of its row; the tiles of grid
  // column pc are owned by chiplet pr*Gc + pc, tn_per_part of them.
  for (int64_t ti = 0; ti < TM; ++ti) {
    std::fill(h.begin(), h.end(), 0);
    ops[OP_A].count(ti * T, (ti + 1) * T, 0, p.K, h.data());
    const int pr = (int)(ti / tm_per_part);
    for (int pc = 0; pc < p.Gc; ++pc) {
      const int o = pr * p.Gc + pc;
      uint64_t rem = ea * (uint64_t)tn_per_part * ((uint64_t)(T * p.K) - h[o]);
      t.remote[OP_A] += rem;
      t.remote_per_chiplet[o] += rem;
    }
  }
  // B: column panel tj is read by the TM tiles of its column.
  for (int64_t tj = 0; tj < TN; ++tj) {
    std::fill(h.begin(), h.end(), 0);
    ops[OP_B].count(0, p.K, tj * T, (tj + 1) * T, h.data());
    const int pc = (int)(tj / tn_per_part);
    for (int pr = 0; pr < p.Gr; ++pr) {
      const int o = pr * p.Gc + pc;
      uint64_t rem = eb * (uint64_t)tm_per_part * ((uint64_t)(p.K * T) - h[o]);
      t.remote[OP_B] += rem;
      t.remote_per_chiplet[o] += rem;
    }
  }
  // C: each tile written once by its owner (and read once before that when
  // c_times == 2; the read has the write's partitioning).
  for (int64_t ti = 0; ti < TM; ++ti) {
    for (int64_t tj = 0; tj < TN; ++tj) {
      std::fill(h.begin(), h.end(), 0);
      ops[OP_C].count(ti * T, (ti + 1) * T, tj * T, (tj + 1) * T, h.data());
      const int o = p.owner(ti, tj);
      uint64_t rem = c_times * ec * ((uint64_t)(T * T) - h[o]);
      t.remote[OP_C] += rem;
      t.remote_per_chiplet[o] += rem;
    }
  }
  t.accessed[OP_A] = ea * (uint64_t)p.M * p.K * TN;
  t.accessed[OP_B] = eb * (uint64_t)p.K * p.N * TM;
  t.accessed[OP_C] = c_times * ec * (uint64_t)p.M * p.N;
  t.floor_bytes = floor_bytes(p.M, p.N, p.K, p.Gr, p.Gc, (int)ea, (int)eb);
  return t;
}

TileMap tile_map(const Plan& p, int splits) {
  const GemmConfig& g = p.gemm;
  const int64_t per_xcd = (g.tiles_m * g.tiles_n * splits + g.xcd_per_chiplet - 1) / g.xcd_per_chiplet;
  return make_tile_map(g.xcd_per_chiplet, p.Gc, (int32_t)g.tiles_m, (int32_t)g.tiles_n,
                 (int32_t)per_xcd, g.group_m, splits);
}

TileMap wide_tile_map(const Plan& p) {
  const GemmConfig& g = p.gemm;
  const int64_t tm = p.part_rows() / 128, tn = p.part_cols() / g.wide_n;
  return make_tile_map(g.xcd_per_chiplet, p.Gc, (int32_t)tm, (int32_t)tn,
                 (int32_t)((tm * tn + g.xcd_per_chiplet - 1) / g.xcd_per_chiplet),
                 (int32_t)std::min<int64_t>(g.wide_group_m, tm), 1);
}

int64_t gemm_ksteps(const Plan& p) {
  return p.K / (p.ab_type == DT_FP8_E4M3 ? kGemmBK8 : kGemmBK);
}

int recommended_splits(const Plan& p) {
  const GemmConfig& g = p.gemm;
  if (!g.supported) return 1;
  // Fill the XCD's 32 CUs when its partition has few tiles, keeping at
  // least 8 K steps per split.
  const int64_t per_xcd = g.tiles_per_xcd;
  int s = (int)std::max<int64_t>(1, 32 / std::max<int64_t>(1, per_xcd));
  s = (int)std::min<int64_t>(s, std::max<int64_t>(1, gemm_ksteps(p) / 8));
  return std::min(s, kMaxSplits);
}

int effective_splits(const Plan& p, int splits) {
  const int64_t ks = gemm_ksteps(p);
  if (splits <= 1 || ks <= 1) return 1;
  const int64_t per = (ks + splits - 1) / splits;
  return (int)((ks + per - 1) / per);
}

int64_t splitk_workgroups(const Plan& p, int splits) {
  const GemmConfig& g = p.gemm;
  const int64_t tiles = g.tiles_m * g.tiles_n * effective_splits(p, splits);
  return kNumXcd * ((tiles + g.xcd_per_chiplet - 1) / g.xcd_per_chiplet);
}

int64_t splitk_reduce_workgroups(const Plan& p) {
  const GemmConfig& g = p.gemm;
  return g.workgroups * (g.tile_m * g.tile_n / 1024);
}

int64_t splitk_workspace_bytes(const Plan& p, int splits) {
  const GemmConfig& g = p.gemm;
  const int s = effective_splits(p, splits);
  return s > 1 ? (int64_t)p.G * g.tiles_m * g.tiles_n * s * g.tile_m * g.tile_n * 4 : 0;
}

static void tile_of(const Plan& p, const TileMap& map, int64_t workgroups, int64_t wg, int* xcd,
                    int64_t* tile_m, int64_t* tile_n) {
  *xcd = (int)(wg % kNumXcd);
  *tile_m = *tile_n = -1;
  int32_t pr, pc, ti, tj;
  if (wg < 0 || wg >= workgroups || !map_tile(map, wg, &pr, &pc, &ti, &tj)) return;
  *tile_m = (int64_t)pr * map.tiles_m + ti;
  *tile_n = (int64_t)pc * map.tiles_n + tj;
}

void tile_of_wg(const Plan& p, int64_t wg, int* xcd, int64_t* tile_m, int64_t* tile_n) {
  tile_of(p, tile_map(p), p.gemm.workgroups, wg, xcd, tile_m, tile_n);
}

void launch_tile_of_wg(const Plan& p, int64_t wg, int* xcd, int64_t* tile_m, int64_t* tile_n) {
  OperandAddr a, b, c;
  ccl_addressing(p, &a, &b, &c);
  const GemmForm f = gemm_form(p, a, b, true, 1);
  tile_of(p, f.map, f.workgroups, wg, xcd, tile_m, tile_n);
}

// A block (pr, kc) = pr*Gc + kc; B block (kr, pc) = kr*Gc + pc; C block (pr, pc).
void ccl_addressing(const Plan& p, OperandAddr* a, OperandAddr* b, OperandAddr* c) {
  const int64_t sa = p.lay[OP_A].strip_stride_bytes / p.lay[OP_A].elem_bytes;
  const int64_t sb = p.lay[OP_B].strip_stride_bytes / p.lay[OP_B].elem_bytes;
  const int64_t sc = p.lay[OP_C].strip_stride_bytes / p.lay[OP_C].elem_bytes;
  *a = {p.Gc * sa, sa, (int32_t)(p.K / p.Gc), (int32_t)(p.K / p.Gc)};
  *b = {sb, p.Gc * sb, (int32_t)(p.N / p.Gc), (int32_t)(p.K / p.Gr)};
  *c = {p.Gc * sc, sc, (int32_t)(p.N / p.Gc), 0};
}

void rowmajor_addressing(const Plan& p, OperandAddr* a, OperandAddr* b, OperandAddr* c) {
  const int64_t hr = p.M / p.Gr;
  *a = {hr * p.K, p.K / p.Gc, (int32_t)p.K, (int32_t)(p.K / p.Gc)};
  *b = {p.N / p.Gc, (p.K / p.Gr) * p.N, (int32_t)p.N, (int32_t)(p.K / p.Gr)};
  *c = {hr * p.N, p.N / p.Gc, (int32_t)p.N, 0};
}

const char* kernel_name(GemmKernel k) {
  switch (k) {
    case GemmKernel::K32: return "gemm_kernel";
    case GemmKernel::K64: return "gemm_k64_kernel";
    case GemmKernel::A2: return "gemm_a2_kernel";
    case GemmKernel::FP8: return "gemm_fp8_kernel";
    case GemmKernel::FP8S: return "gemm_fp8s_kernel";
    case GemmKernel::FP8X: return "gemm_fp8x_kernel";
    case GemmKernel::FP8P: return "gemm_fp8p_kernel";
  }
  return "";
}

GemmForm gemm_form(const Plan& p, const OperandAddr& a, const OperandAddr& b, bool remap, int splits,
                   bool reads_c) {
  const GemmConfig& g = p.gemm;
  const bool fp8 = p.ab_type == DT_FP8_E4M3;
  const int64_t e = fp8 ? 1 : 2;
  const bool full = g.tile_m == 256 && g.tile_n == 256;
  GemmForm f;
  f.splits = effective_splits(p, splits);      // every K range non-empty
  f.tile_m = g.tile_m;
  f.tile_n = g.tile_n;
  f.waves = g.waves;
  f.map = tile_map(p, f.splits);
  f.ksteps = (int32_t)gemm_ksteps(p);
  f.ksteps_per_split = (f.ksteps + f.splits - 1) / f.splits;
  // Non-temporal stores of C: always for a bf16 C of the pipelined fp8 kernel
  // (1-4 % faster at the power limit) and where B streams; elsewhere, for a bf16
  // C of the 64- and 128-K-stage kernels, where operands and C together exceed
  // the Infinity Cache. Below that what reads C next (the unpack or the next
  // GEMM) finds it in the cache, and the operands stay too: whole passes of
  // pack, GEMM and unpack, non-temporal -> plain, 4096x1536x2048 42.1 -> 40.2 us,
  // 4096x768x2048 29.2 -> 28.4, 256x512x256 10.7 -> 10.4, while the launch alone
  // takes 0-12 % longer. Above it plain stores push the operands out:
  // 640x16384x7168 161.5 -> 172.6, 384x28672x4096 105.4 -> 111.1.
  // Row-major C in native tile order (each XCD writes stretches of every row)
  // always goes past the cache: the launch alone 4480x5120x512 40.8 -> 33.5 us,
  // 1920x14336x256 37.3 -> 32.0, with a reader behind it 55.5 -> 51.1 and 52.9 ->
  // 51.6, up to 12 MB 0-5 % longer.
  // An fp32 C, in every kernel, from the cache's size on: 2048x4096x1024 39.4 ->
  // 36.1, 5888x1024x1024 36.1 -> 33.5, but fp8 8192x8192x1024 (256 MiB) 176 -> 192.
  f.c_nt = p.c_type == DT_FP32 ? p.M * p.N * 4 >= kInfinityCacheBytes
                               : !remap || (p.M * p.K + p.K * p.N) * e + p.M * p.N * 2 > kInfinityCacheBytes;
  const auto set_grid = [&] {
    f.workgroups = remap ? 8 * (int64_t)f.map.tiles_per_xcd : (int64_t)f.map.tiles_m * f.map.tiles_n * p.G;
  };
  set_grid();
  // One descriptor per operand for a tile over all K blocks: both extents
  // within the 31 bits of its offsets.
  const int64_t lim = ((int64_t)1 << 31) - 4096;
  const bool fits = ((p.K / a.kslice - 1) * a.slice + 256 * (int64_t)a.ld) * e < lim &&
                    ((p.K / b.kslice - 1) * b.slice + (int64_t)b.kslice * b.ld + 256) * e < lim;
  // Steps of bk (twice the plan's), and whether they lie in one K block each
  // and cut K into the same ranges: the workspace and the reduce do not
  // depend on the kernel.
  const auto whole_steps = [&](int bk, int32_t* steps, int32_t* per) {
    *steps = (int32_t)(p.K / bk);
    *per = (*steps + f.splits - 1) / f.splits;
    return a.kslice % bk == 0 && b.kslice % bk == 0 && (f.splits == 1 || 2 * *per == f.ksteps_per_split);
  };
  int32_t steps, per;
  if (fp8) {
    const bool whole = whole_steps(kGemmBK8x, &steps, &per);
    // More than 32 split-K workgroups of 128x128 per XCD run the 32x32x64 kernel,
    // two to a CU: short K ranges and fp32 stores wait on memory. Us, 128-K
    // stages -> it: 9 tiles, K 2048, in 4 ranges 14.1 -> 12.9 (in 2 11.1 -> 11.5),
    // 25 tiles in 2 ranges 21.6 -> 20.6, 63 tiles, K 4096, in 2 63.0 -> 53.7, in 4
    // 77.0 -> 68.5. So do unsplit launches that write an fp32 C without reading
    // it, up to K 2048: pack, GEMM and unpack, 63 tiles, K 256 31.0 -> 28.5, K 1024
    // 37.1 -> 33.3, 273 tiles, K 2048 168 -> 155 (45 tiles 37.0 -> 38.0). With a
    // bf16 C they gain up to 15 % from 128-K stages, or lose 3 % at 33 tiles, and
    // with an fp32 C that is read 4-29 %.
    const bool partials = f.splits > 1 || (p.c_type == DT_FP32 && !reads_c && p.K <= 2048);
    const bool paired = partials && g.tile_m == 128 && g.tile_n == 128 && f.map.tiles_per_xcd > 32;
    // 256x256 tiles with 8 waves: the 16x16x128 kernels (no split-K), the
    // pipelined one where its descriptors reach. Below 256x256 (8 waves, the
    // plan's choice where both K blocks are multiples of 128): 128-K stages.
    // Other plans run the 32x32x64 kernel.
    if (full && f.splits == 1 && g.waves == 8 && whole) {
      f.kernel = g.fp8_pipe && fits ? GemmKernel::FP8P : GemmKernel::FP8X;
    } else if (!full && g.waves == 8 && whole && fits && !paired) {
      f.kernel = GemmKernel::FP8S;
    } else {
      f.kernel = GemmKernel::FP8;
      if (!full) f.waves = 4;
      return f;
    }
    f.ksteps = steps;
    f.ksteps_per_split = per;
    return f;
  }
  const bool whole = whole_steps(kGemmBK64, &steps, &per);
  // 128x192 or 128x320 tiles: the plan's choice for unsplit launches under the
  // XCD-aware map, with operands that fit.
  const bool wide = g.wide_n && remap && f.splits == 1 && fits && !g.far;
  if (wide) {
    f.tile_m = 128;
    f.tile_n = g.wide_n;
    f.map = wide_tile_map(p);
    set_grid();
  }
  // 64-K stages (the plan's choice for the bf16 tiles below 256x256). Where
  // both K blocks are multiples of 64 and split-K cuts K at whole stages, a
  // stage lies in one K block, and operands of 2 GiB and more take the far
  // form; otherwise the ragged form, whose K ranges are the 32-K ranges, whose
  // K blocks hold at least a stage and whose extents fit in 31 bits.
  // The ragged form adds to A's addresses what the next K block takes, which
  // must pay for itself (us per launch, 32-K stages -> ragged 64-K ones):
  //  * 128x128, up to 32 tiles per XCD, one per CU: it does (18 tiles,
  //    1152x2048x3328: 27.4 -> 26.5; 24, 1024x3072x9984: 104.6 -> 88.3). Above
  //    32, two workgroups of 32-K stages (64 KiB) share a CU: 33 to 105 tiles
  //    take 6-25 % longer with 64-K stages at K up to 1056, the same at 2080
  //    and 0-6 % less at 4128.
  //  * 256x128: from about 2048 K on (24 tiles: K 544 11.5 -> 12.3, 1056 17.1
  //    -> 17.9, 2080 30.8 -> 29.0, 4128 57.5 -> 52.7; 33 tiles: 22.1 -> 22.9,
  //    34.8 -> 33.8, 60.7 -> 56.3, 118 -> 106).
  //  * 128x256: not (8 to 90 tiles, K 224 to 8224: 0-10 % longer), unless the
  //    operands exceed the Infinity Cache, where whole lines count (33 to 90
  //    tiles, 3 to 9 tile rows of 22528, K 8448: 241 -> 220, 281 -> 242).
  //  * not where only the K ranges are odd: every second one starts in the middle
  //    of A's 128-byte lines (2 to 9 tiles, K 6016 in 3 ranges of 63 steps: 20.5
  //    -> 21.6, 24.1 -> 25.2).
  const bool blocks_whole = a.kslice % kGemmBK64 == 0 && b.kslice % kGemmBK64 == 0;
  const int64_t range_k = (int64_t)f.ksteps_per_split * kGemmBK;
  const bool ragged_pays =
      !blocks_whole &&
      (g.tile_n == 256   ? (p.M + p.N) * p.K * e > kInfinityCacheBytes
       : g.tile_m == 256 ? range_k >= 1536
                         : f.map.tiles_per_xcd <= 32);
  const bool exists = whole || (fits && a.kslice >= kGemmBK64 && b.kslice >= kGemmBK64);
  if (wide || (g.stage_k == 64 && g.waves == 8 && !full && exists && (whole || ragged_pays || g.stage_64))) {
    f.kernel = GemmKernel::K64;
    f.ragged = !whole;
    f.far = whole && (!fits || g.far);
    f.stream_b = g.stream_b && remap && f.map.tiles_m == 1;
    if (whole) {
      f.ksteps = steps;
      f.ksteps_per_split = per;
    }
    return f;
  }
  // The 64-K-pair kernel's A descriptor spans the tile's 256 rows over all
  // K blocks of A.
  if (g.a_pairs && f.splits == 1 && g.waves == 8 && full && a.kslice % kGemmBK64 == 0 &&
      (p.K / a.kslice - 1) * a.slice * 2 + 256 * (int64_t)a.ld * 2 + 4096 < ((int64_t)1 << 31))
    f.kernel = GemmKernel::A2;
  return f;
}

}  // namespace ccl
