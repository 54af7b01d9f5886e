// Pack / unpack between row-major (or stored-transpose) operands and the
// Chiplet-Contiguous Layout (Sec. III-B, Eq. 3 in block form); elements of
// 1, 2 or 4 bytes (fp8, bf16, fp32) are moved as bits:
//   block b = (r / hr) * Gc + c / wc
//   byte offset = b * S + ((r % hr) * wc + c % wc) * e     (S = padded strip)
//
// The work is enumerated in CCL order: block b, then its q-th element (or
// 16-byte chunk) in strip order, so every thread's CCL access is the next
// contiguous piece of a strip and its row-major access is a contiguous run
// of one row slice. Division by the run length uses a host-computed
// multiplier. These kernels move bytes only; they are bound by HBM.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "kernels.hpp"

namespace ccl {

namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));   // one 16-byte chunk

// Workgroups of copy_stream_kernel's resident grid: 8 of 256 threads per CU
// on 256 CUs (2048 measured best of 1024, 2048, 3072 and 4096).
constexpr unsigned kResidentWgs = 2048;

// q / d for q < 2^31, d < 2^31: multiply by ceil(2^s / d), s = 31 + ceil(log2 d).
struct DivMagic {
  uint64_t mul;
  uint32_t shift;
  uint32_t d;
};

DivMagic make_div(uint32_t d) {
  uint32_t l = 0;
  while ((1ull << l) < d) ++l;
  DivMagic m;
  m.shift = 31 + l;
  m.mul = (((uint64_t)1 << m.shift) + d - 1) / d;
  m.d = d;
  return m;
}

__device__ __forceinline__ uint32_t fdiv(uint32_t q, const DivMagic& m) {
  return (uint32_t)(((uint64_t)q * m.mul) >> m.shift);
}

struct PackArgs {
  const char* rm;          // row-major side
  char* rm_out;            // row-major side when written (unpack)
  const char* ccl;         // CCL side (read by unpack)
  char* ccl_out;           // CCL side (written by pack)
  int64_t ld_bytes;        // row-major leading dimension
  int64_t strip;           // padded strip stride, bytes
  int64_t hr;              // block rows
  int64_t row_bytes;       // bytes of one block row (wc * e)
  int32_t grid_c;
  uint32_t units_per_block;  // hr * units_per_row
  DivMagic units_per_row;    // ceil(row_bytes / unit)
};

// Byte offsets of unit q of a block on both sides. Units are US bytes of one
// block row. EXACT: a row is a whole number of them. Otherwise its last unit
// ends at the row's end and overlaps the one before (the same bytes twice),
// so no access leaves the row.
template <int64_t US, bool EXACT>
__device__ __forceinline__ void unit_offsets(const PackArgs& a, uint32_t q, int64_t* rm, int64_t* ccl) {
  const uint32_t row = fdiv(q, a.units_per_row);
  const uint32_t i = q - row * a.units_per_row.d;
  int64_t col = (int64_t)i * US;
  if constexpr (!EXACT) col = std::min<int64_t>(col, a.row_bytes - US);
  *rm = (int64_t)row * a.ld_bytes + col;
  *ccl = EXACT ? (int64_t)q * US : (int64_t)row * a.row_bytes + col;
}

// Load / store one unit of type T; NT = non-temporal (streaming) access; ANY:
// at any byte address, which gfx950 global accesses take in one instruction
// like an aligned one. (A typedef of its own here: a template argument would
// lose the attribute.)
template <typename T, bool NT, bool ANY>
__device__ __forceinline__ T ld(const char* p) {
  typedef T any __attribute__((aligned(1)));
  static_assert(alignof(any) == 1, "the compiler may not assume an alignment");
  if constexpr (ANY && NT) return __builtin_nontemporal_load(reinterpret_cast<const any*>(p));
  else if constexpr (ANY) return *reinterpret_cast<const any*>(p);
  else if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const T*>(p));
  else return *reinterpret_cast<const T*>(p);
}
template <typename T, bool NT, bool ANY>
__device__ __forceinline__ void st(char* p, T v) {
  typedef T any __attribute__((aligned(1)));
  if constexpr (ANY && NT) __builtin_nontemporal_store(v, reinterpret_cast<any*>(p));
  else if constexpr (ANY) *reinterpret_cast<any*>(p) = v;
  else if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<T*>(p));
  else *reinterpret_cast<T*>(p) = v;
}

// Tensors above the Infinity Cache size, with streaming (non-temporal) loads
// and stores (measured: +10 % on a 470 MB copy, -15 % on a 134 MB one that
// the cache holds; NT = false: plain accesses). U = unit moved per access, at
// any byte address: 16 bytes, or one element. UNPACK = false: row-major -> CCL;
// true: CCL -> row-major.
template <typename U, bool UNPACK, bool EXACT, bool NT>
__global__ void __launch_bounds__(256) copy_kernel(PackArgs a) {
  const int32_t b = blockIdx.y;                      // strip / chiplet
  const int64_t pr = b / a.grid_c, pc = b % a.grid_c;
  const int64_t rm_base = pr * a.hr * a.ld_bytes + pc * a.row_bytes;
  const char* src = UNPACK ? a.ccl + (int64_t)b * a.strip : a.rm + rm_base;
  char* dst = UNPACK ? a.rm_out + rm_base : a.ccl_out + (int64_t)b * a.strip;
  constexpr int UNROLL = 4;
  const uint32_t stride = gridDim.x * 256u;
  for (uint32_t base = blockIdx.x * 256u * UNROLL; base < a.units_per_block; base += stride * UNROLL) {
    U v[UNROLL];
    int64_t to[UNROLL];
    bool ok[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const uint32_t q = base + threadIdx.x + u * 256u;
      ok[u] = q < a.units_per_block;
      int64_t rm, ccl;
      unit_offsets<sizeof(U), EXACT>(a, q, &rm, &ccl);
      to[u] = UNPACK ? rm : ccl;
      if (ok[u]) v[u] = ld<U, NT, true>(src + (UNPACK ? ccl : rm));
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u)
      if (ok[u]) st<U, NT, true>(dst + to[u], v[u]);
  }
}

// Tensors below the Infinity Cache size: a resident grid
// (about 8 workgroups per CU) walks each strip with a stride of the whole
// grid, and issues the loads of its next round before the stores of the
// current one, so every workgroup keeps a round of loads in flight instead
// of one load-then-store pass per workgroup. Loads stream (the source is
// not read again by the path); stores are plain, so the packed operand can
// stay in the Infinity Cache for the GEMM that reads it next (streaming
// stores made the 134 MB activation pack 12 % slower between the FFN GEMMs).
// Measured on the 134 MB pack of X from HBM: 5.39-5.41 TB/s against
// 5.05-5.14 for copy_kernel; inside the FFN step 46 us against 54 us. U as
// in copy_kernel.
template <typename U, bool UNPACK, bool EXACT, int UNROLL>
__global__ void __launch_bounds__(256) copy_stream_kernel(PackArgs a) {
  const int32_t b = blockIdx.y;                      // strip / chiplet
  const int64_t pr = b / a.grid_c, pc = b % a.grid_c;
  const int64_t rm_base = pr * a.hr * a.ld_bytes + pc * a.row_bytes;
  const char* src = UNPACK ? a.ccl + (int64_t)b * a.strip : a.rm + rm_base;
  char* dst = UNPACK ? a.rm_out + rm_base : a.ccl_out + (int64_t)b * a.strip;
  constexpr uint32_t kRound = 256u * UNROLL;         // units per workgroup round
  const uint32_t stride = gridDim.x * kRound;
  auto load = [&](uint32_t base, U* v) {
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const uint32_t q = base + threadIdx.x + u * 256u;
      if (q < a.units_per_block) {
        int64_t rm, ccl;
        unit_offsets<sizeof(U), EXACT>(a, q, &rm, &ccl);
        v[u] = ld<U, true, true>(src + (UNPACK ? ccl : rm));
      }
    }
  };
  auto store = [&](uint32_t base, const U* v) {
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const uint32_t q = base + threadIdx.x + u * 256u;
      if (q < a.units_per_block) {
        int64_t rm, ccl;
        unit_offsets<sizeof(U), EXACT>(a, q, &rm, &ccl);
        st<U, false, true>(dst + (UNPACK ? rm : ccl), v[u]);
      }
    }
  };
  uint32_t base = blockIdx.x * kRound;
  if (base >= a.units_per_block) return;
  U cur[UNROLL], nxt[UNROLL];
  load(base, cur);
  for (; base < a.units_per_block; base += stride) {
    const uint32_t next = base + stride;
    if (next < a.units_per_block) load(next, nxt);
    store(base, cur);
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) cur[u] = nxt[u];
  }
}

// Stored-transpose packs: src holds X^T (cols x rows, leading dimension ld
// elements), X is rows x cols of element type E.
struct TransArgs {
  const char* src;
  char* dst;
  int64_t ld;              // elements
  int64_t strip;           // bytes
  int64_t hr, wc;          // elements
  int32_t grid_c;
  int32_t rows, cols;
  DivMagic div_hr, div_wc;
};

// One element per thread, for small tensors, which wait on latency alone.
template <typename E>
__global__ void __launch_bounds__(256) pack_trans_scalar_kernel(TransArgs a, DivMagic div_cols) {
  const uint32_t n = (uint32_t)a.rows * (uint32_t)a.cols;
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i < n) {
    const uint32_t r = fdiv(i, div_cols), c = i - r * div_cols.d;      // write order: along X rows
    const uint32_t pr = fdiv(r, a.div_hr), pc = fdiv(c, a.div_wc);
    char* strip = a.dst + ((int64_t)pr * a.grid_c + pc) * a.strip;
    st<E, false, true>(strip + ((r - pr * a.hr) * a.wc + (c - pc * a.wc)) * (int64_t)sizeof(E),
                       ld<E, false, true>(a.src + (c * a.ld + r) * (int64_t)sizeof(E)));
  }
}

// fp8 through LDS, for blocks whose sides are multiples of 64 but not of the
// register kernel's 128 below, and 16-byte aligned operands. A 64 x 64 tile is
// read along X's rows (contiguous in src) in 16-byte chunks, transposed through
// LDS and written in 16-byte chunks along X's columns. Tiles never straddle
// blocks.
__global__ void __launch_bounds__(256) pack_trans_lds_kernel(TransArgs a) {
  __shared__ uint8_t tile[64][64 + 16];
  const int64_t r0 = (int64_t)blockIdx.y * 64;        // X rows = src columns
  const int64_t c0 = (int64_t)blockIdx.x * 64;        // X cols = src rows
  const int line = threadIdx.x / 4, ch = threadIdx.x % 4;
  const u32x4 in = ld<u32x4, false, false>(a.src + (c0 + line) * a.ld + r0 + ch * 16);
  *reinterpret_cast<u32x4*>(&tile[line][ch * 16]) = in;
  __syncthreads();
  const int64_t pr = r0 / a.hr, pc = c0 / a.wc;
  char* strip = a.dst + (pr * a.grid_c + pc) * a.strip;
  u32x4 out;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    uint32_t w = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) w |= (uint32_t)tile[ch * 16 + 4 * q + j][line] << (8 * j);
    out[q] = w;
  }
  st<u32x4, false, false>(strip + (r0 - pr * a.hr + line) * a.wc + (c0 - pc * a.wc) + ch * 16, out);
}

// Stored-transpose pack without LDS. With EPC elements per 16-byte chunk,
// each thread moves an EPC x EPC block: it reads EPC chunks, one from each
// of EPC consecutive rows of the stored transpose, transposes the block in
// registers (byte permutes) and writes EPC chunks along consecutive rows of
// the CCL strip. Lane (a, b) = (lane % 8, lane / 8) covers X rows
// R0 + EPC a .. + EPC - 1 and X columns C0 + EPC b .. + EPC - 1, so a wave
// covers a WB x WB block (WB = 8 EPC) and each of its loads and stores
// touches 8 rows x 128 contiguous bytes. The 4 waves of a workgroup take 4
// consecutive blocks along X's columns. Loads stream: the stored tensor is
// read once (134 MB from HBM: 5.05 against 4.92 TB/s). NTS: streaming stores,
// for operands above the Infinity Cache size (470 MB W_up^T: 162 against
// 177 us with plain ones). Below it they are plain, so the GEMM that follows
// finds the operand in the cache: alone, the 134 MB transpose is 12 % faster
// with streaming stores, but the whole weight-gradient pass is not (2943
// against 2938 us), and at 6 MB the GEMM behind the pack took 41 us instead
// of 29 (pass 55.3 against 42.9 us; 768x2048x4096: 43.6 against 37.4).
// RAGGED = false: hr and wc are multiples of WB, so a wave's block never
// straddles CCL blocks, and src and dst are 16-byte aligned. RAGGED = true:
// hr and wc are multiples of EPC only, so each thread's own EPC x EPC block
// lies within one CCL block, which it finds for itself; any alignment. Against
// one element per thread: 1152x3328 bf16 in 416-column blocks 19.4 -> 5.0 us
// (odd leading dimension 20.7 -> 6.4), 4096x2112 fp8 37.0 -> 7.4.
template <typename E, bool RAGGED, bool NTS>
__global__ void __launch_bounds__(256) pack_trans_reg_kernel(TransArgs a, int32_t wb_cols, int32_t y0) {
  constexpr int EPC = 16 / (int)sizeof(E);
  constexpr int WB = 8 * EPC;
  typedef E ev __attribute__((ext_vector_type(EPC)));
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  // Row block by of column group bx: y0 (of a launch of at most 65535 row
  // blocks) plus blockIdx.y skewed by 2 blocks per column group, so that the workgroups resident at one time read chunks
  // spread over the width of the stored rows instead of one 8 KiB band of
  // them (a bijection for each bx). Measured from HBM against no skew:
  // 134 MB X^T 0.663-0.666 of 8 TB/s against 0.627-0.628, 470 MB W_up^T
  // 0.710 against 0.698-0.699; skews of 1, 3 and 4 were 0-1 % slower, 8
  // and 16 (several column groups then share a band) 4 % and 20 % slower.
  const int32_t bx = blockIdx.x, by = y0 + (int32_t)((blockIdx.y + blockIdx.x * 2u) % gridDim.y);
  const int32_t wcb = bx * 4 + wave;
  if (wcb >= wb_cols) return;
  const int la = lane & 7, lb = lane >> 3;
  const int64_t R0 = (int64_t)by * WB, C0 = (int64_t)wcb * WB;
  if constexpr (RAGGED)
    if (R0 + EPC * la >= a.rows || C0 + EPC * lb >= a.cols) return;
  const E* src = reinterpret_cast<const E*>(a.src) + (C0 + EPC * lb) * a.ld + R0 + EPC * la;
  ev in[EPC];
#pragma unroll
  for (int j = 0; j < EPC; ++j)
    in[j] = __builtin_bit_cast(ev, ld<u32x4, true, RAGGED>(reinterpret_cast<const char*>(src + j * a.ld)));
  const uint32_t r = (uint32_t)R0 + (RAGGED ? EPC * la : 0), c = (uint32_t)C0 + (RAGGED ? EPC * lb : 0);
  const uint32_t pr = fdiv(r, a.div_hr), pc = fdiv(c, a.div_wc);
  E* strip = reinterpret_cast<E*>(a.dst + ((int64_t)pr * a.grid_c + pc) * a.strip);
  E* dst = strip + (R0 - pr * a.hr + EPC * la) * a.wc + (C0 - pc * a.wc) + EPC * lb;
#pragma unroll
  for (int i = 0; i < EPC; ++i) {
    ev o;
#pragma unroll
    for (int j = 0; j < EPC; ++j) o[j] = in[j][i];
    st<u32x4, NTS, RAGGED>(reinterpret_cast<char*>(dst + i * a.wc), __builtin_bit_cast(u32x4, o));
  }
}

// Any shape: a 64 x 64 tile through LDS, element by element, so that both
// the reads (along X's rows, contiguous in src) and the writes (along X's
// columns, contiguous in a block) of a wave cover whole lines: 8192x8200 bf16
// in 1025-column blocks 355 -> 116 us against one element per thread.
template <typename E>
__global__ void __launch_bounds__(256) pack_trans_any_kernel(TransArgs a, uint32_t row_tiles,
                                                             uint32_t tiles) {
  __shared__ E tile[64][64 + 4 / sizeof(E)];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (uint32_t t = blockIdx.x; t < tiles; t += gridDim.x) {
    const uint32_t tc = t / row_tiles, tr = t - tc * row_tiles;
    const int64_t r0 = (int64_t)tr * 64, c0 = (int64_t)tc * 64;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int c = i * 4 + wave;
      if (r0 + lane < a.rows && c0 + c < a.cols)
        tile[c][lane] = ld<E, false, true>(a.src + ((c0 + c) * a.ld + r0 + lane) * (int64_t)sizeof(E));
    }
    __syncthreads();
    const int64_t col = c0 + lane;
    if (col < a.cols) {
      const uint32_t pc = fdiv((uint32_t)col, a.div_wc);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int64_t row = r0 + i * 4 + wave;
        if (row >= a.rows) continue;
        const uint32_t pr = fdiv((uint32_t)row, a.div_hr);
        char* strip = a.dst + ((int64_t)pr * a.grid_c + pc) * a.strip;
        st<E, false, true>(strip + ((row - pr * a.hr) * a.wc + col - pc * a.wc) * (int64_t)sizeof(E),
                           tile[lane][i * 4 + wave]);
      }
    }
    __syncthreads();
  }
}

int grid_x_for(uint32_t units, int unroll) {
  uint64_t wgs = ((uint64_t)units + 256ull * unroll - 1) / (256ull * unroll);
  if (wgs > 4096) wgs = 4096;
  return (int)(wgs ? wgs : 1);
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

template <typename U, bool UNPACK, int UNROLL>
void copy_stream_launch(dim3 grid, const PackArgs& a, bool exact, hipStream_t stream) {
  if (exact)
    hipLaunchKernelGGL((copy_stream_kernel<U, UNPACK, true, UNROLL>), grid, dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL((copy_stream_kernel<U, UNPACK, false, UNROLL>), grid, dim3(256), 0, stream, a);
}

template <typename U, bool UNPACK>
void copy_launch_as(dim3 grid, const PackArgs& a, bool big, int unroll, bool exact, hipStream_t stream) {
  if (big && exact)
    hipLaunchKernelGGL((copy_kernel<U, UNPACK, true, true>), grid, dim3(256), 0, stream, a);
  else if (big)
    hipLaunchKernelGGL((copy_kernel<U, UNPACK, false, true>), grid, dim3(256), 0, stream, a);
  else if (unroll == 1)
    copy_stream_launch<U, UNPACK, 1>(grid, a, exact, stream);
  else if (unroll == 2)
    copy_stream_launch<U, UNPACK, 2>(grid, a, exact, stream);
  else
    copy_stream_launch<U, UNPACK, 4>(grid, a, exact, stream);
}

// Units of type U: fills in the unit counts and picks the kernel by size.
template <typename U>
void copy_launch(const Layout& L, PackArgs a, bool unpack, hipStream_t stream) {
  const int64_t per_row = (a.row_bytes + (int64_t)sizeof(U) - 1) / (int64_t)sizeof(U);
  const bool exact = per_row * (int64_t)sizeof(U) == a.row_bytes;
  a.units_per_block = (uint32_t)(L.block_rows * per_row);
  a.units_per_row = make_div((uint32_t)per_row);
  const unsigned strips = (unsigned)(L.grid_r * L.grid_c);
  // above the cache size both sides stream (measured: +10 % on 470 MB);
  // below it a resident grid: kResidentWgs workgroups in all, at most one
  // round each per strip. Where that grid holds the whole tensor at one or two
  // units per thread, threads take that many instead of four: such copies wait
  // on latency, and four units per thread left half or more of the CUs without
  // a workgroup. Whole passes of pack, GEMM and unpack: 256x512x256 10.4 -> 9.5
  // us, 4096x1536x2048 44.1 -> 42.9, in fp8 32.6 -> 30.8, 4096x768x2048 30.3 -> 29.9.
  const bool big = L.rows * L.cols * L.elem_bytes > kInfinityCacheBytes;
  const unsigned resident = std::max(1u, kResidentWgs / strips);
  // One unit per thread up to three quarters of the grid only: packs of 6.5 to
  // 8 MB take 3-4 % less with two.
  const int unroll = big ? 4 : a.units_per_block <= resident * 192ull ? 1 : a.units_per_block <= resident * 512ull ? 2 : 4;
  dim3 grid(grid_x_for(a.units_per_block, unroll), strips);
  if (!big) grid.x = std::min(resident, grid.x);
  if (unpack) copy_launch_as<U, true>(grid, a, big, unroll, exact, stream);
  else copy_launch_as<U, false>(grid, a, big, unroll, exact, stream);
}

// aligned: src, ld, dst and strips are multiples of 16 bytes.
template <typename E>
void trans_launch(const Layout& L, const TransArgs& a, bool aligned, hipStream_t stream) {
  constexpr int EPC = 16 / (int)sizeof(E);
  constexpr int WB = 8 * EPC;         // block edge of a wave of the register kernel
  const int64_t n = L.rows * L.cols;
  const auto blocks_of = [&](int m) { return L.block_rows % m == 0 && L.block_cols % m == 0; };
  const bool whole = aligned && blocks_of(WB), chunks = blocks_of(EPC);
  // Small tensors that the register kernel takes ragged or not at all: few of
  // its waves, or of the tiles, wait out 16 / sizeof(E) or 16 loads in turn. Us,
  // one element per thread -> register blocks or tiles: fp8 64 Ki elements 2.0
  // -> 3.5, 512 Ki 3.5 -> 3.9 (but 1 Mi 5.8 -> 4.2), bf16 64 Ki 2.0 -> 2.6, 181 Ki
  // 2.3 -> 2.8 (362 Ki 3.3 -> 2.9), fp32 tiles 64 Ki 2.0 -> 4.4, 724 Ki 4.6 -> 5.6
  // (1448 Ki 10.5 -> 6.8); fp32 register blocks are as fast from the start.
  const int64_t small = !chunks ? 7 << 17 : sizeof(E) == 1 ? 11 << 16 : sizeof(E) == 2 ? 1 << 18 : 0;
  if (!whole && !(sizeof(E) == 1 && aligned && blocks_of(64)) && n <= small) {
    hipLaunchKernelGGL((pack_trans_scalar_kernel<E>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, a,
                       make_div((uint32_t)L.cols));
    return;
  }
  if constexpr (sizeof(E) == 1) {
    // Sides of 64 mod 128: 64 x 64 tiles, of which there are four for each wave
    // block, up to 8 MiB. Us, tiles -> ragged register blocks: 64 KiB 2.0 -> 3.1,
    // 1 MiB 2.3 -> 4.0, 4 MiB 3.6 -> 4.5, 8 MiB 5.3 -> 5.4, 14 MiB 7.9 -> 6.8.
    // Above that where the tile columns are a multiple of the 8 XCDs: the two
    // tiles that share each 128-byte line of src then run on one XCD (17 MB in
    // 4608 columns 8.3 -> 11.2, 36 MB in 5120 13.3 -> 17.2, 45 MB in 10240 15.6 ->
    // 18.7, 48 MB in 8192 17.2 -> 19.8; else 25 MB in 7040 13.3 -> 12.5, 60 MB in
    // 12416 28.4 -> 24.3).
    if (!whole && aligned && blocks_of(64) && L.rows / 64 <= 65535 && (n <= 8 << 20 || L.cols % 512 == 0)) {
      hipLaunchKernelGGL(pack_trans_lds_kernel, dim3((unsigned)(L.cols / 64), (unsigned)(L.rows / 64)), dim3(256), 0,
                         stream, a);
      return;
    }
  }
  if (whole || chunks) {
    const int32_t wb_cols = (int32_t)((L.cols + WB - 1) / WB), wb_rows = (int32_t)((L.rows + WB - 1) / WB);
    const bool big = n * (int64_t)sizeof(E) > kInfinityCacheBytes;
    for (int32_t y0 = 0; y0 < wb_rows; y0 += 65535) {
      const dim3 grid((unsigned)((wb_cols + 3) / 4), (unsigned)std::min(wb_rows - y0, 65535));
#define CCL_REG(RAGGED_, NTS_) \
  hipLaunchKernelGGL((pack_trans_reg_kernel<E, RAGGED_, NTS_>), grid, dim3(256), 0, stream, a, wb_cols, y0)
      if (whole && big) CCL_REG(false, true);
      else if (whole) CCL_REG(false, false);
      else if (big) CCL_REG(true, true);
      else CCL_REG(true, false);
#undef CCL_REG
    }
    return;
  }
  const int64_t row_tiles = (L.rows + 63) / 64, tiles = row_tiles * ((L.cols + 63) / 64);
  hipLaunchKernelGGL((pack_trans_any_kernel<E>), dim3((unsigned)std::min<int64_t>(tiles, 1 << 20)),
                     dim3(256), 0, stream, a, (uint32_t)row_tiles, (uint32_t)tiles);
}

}  // namespace

hipError_t launch_copy(const Plan& p, int op, const void* rowmajor, int64_t ld, void* ccl_buf,
                       bool unpack, hipStream_t stream) {
  const Layout& L = p.lay[op];
  const int64_t e = L.elem_bytes;
  PackArgs a;
  a.rm = static_cast<const char*>(rowmajor);
  a.rm_out = const_cast<char*>(static_cast<const char*>(rowmajor));
  a.ccl = static_cast<const char*>(ccl_buf);
  a.ccl_out = static_cast<char*>(ccl_buf);
  a.ld_bytes = ld * e;
  a.strip = L.strip_stride_bytes;
  a.hr = L.block_rows;
  a.row_bytes = L.block_cols * e;
  a.grid_c = (int32_t)L.grid_c;
  // 16-byte units wherever a block row holds one, whatever the alignment.
  // Against one element per access: 8192x8192 bf16 with an odd leading
  // dimension 104 -> 50 us, in rows of 1025 elements 108 -> 60 us (unpack 109
  // -> 63), 4096x2048 12.8 -> 7.6 us.
  // fp32 rows off the 16-byte grid stay at one element per access where both
  // sides fit in the Infinity Cache together but hardly one in the L2s (8 x 4
  // MiB). Us, elements -> units, pack and unpack: 31 MB 13.5 -> 15.9, 40 MB 14.6
  // -> 18.8 and 14.1 -> 18.1, 77 MB 26.5 -> 31.1 and 25.4 -> 31.7, 109 MB 36.0 ->
  // 41.3 and 34.3 -> 41.6; outside, 24 MB 9.8 -> 8.6 and 9.6 -> 8.6, 150 MB 66.6
  // -> 49.0 and 58.9 -> 48.4.
  const int64_t bytes = L.rows * L.cols * e;
  const bool on_grid = (a.row_bytes | a.ld_bytes | a.strip) % 16 == 0 && aligned16(rowmajor) && aligned16(ccl_buf);
  if (e == 4 && !on_grid && bytes > (28 << 20) && 2 * bytes <= kInfinityCacheBytes) {
    a.units_per_block = (uint32_t)(L.block_rows * L.block_cols);
    a.units_per_row = make_div((uint32_t)L.block_cols);
    const dim3 grid(grid_x_for(a.units_per_block, 4), (unsigned)(L.grid_r * L.grid_c));
    if (unpack) hipLaunchKernelGGL((copy_kernel<uint32_t, true, true, false>), grid, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((copy_kernel<uint32_t, false, true, false>), grid, dim3(256), 0, stream, a);
  } else if (a.row_bytes >= 16)
    copy_launch<u32x4>(L, a, unpack, stream);
  else if (e == 1)
    copy_launch<uint8_t>(L, a, unpack, stream);
  else if (e == 2)
    copy_launch<uint16_t>(L, a, unpack, stream);
  else
    copy_launch<uint32_t>(L, a, unpack, stream);
  return hipGetLastError();
}

hipError_t launch_pack_trans(const Plan& p, int op, const void* src, int64_t ld, void* dst,
                             hipStream_t stream) {
  const Layout& L = p.lay[op];
  const int64_t e = L.elem_bytes;
  TransArgs a;
  a.src = static_cast<const char*>(src);
  a.dst = static_cast<char*>(dst);
  a.ld = ld;
  a.strip = L.strip_stride_bytes;
  a.hr = L.block_rows;
  a.wc = L.block_cols;
  a.grid_c = (int32_t)L.grid_c;
  a.rows = (int32_t)L.rows;
  a.cols = (int32_t)L.cols;
  a.div_hr = make_div((uint32_t)L.block_rows);
  a.div_wc = make_div((uint32_t)L.block_cols);
  const bool aligned = (ld * e) % 16 == 0 && aligned16(src) && aligned16(dst) &&
                       L.strip_stride_bytes % 16 == 0;
  if (e == 1)
    trans_launch<uint8_t>(L, a, aligned, stream);
  else if (e == 2)
    trans_launch<uint16_t>(L, a, aligned, stream);
  else
    trans_launch<uint32_t>(L, a, aligned, stream);
  return hipGetLastError();
}

}  // namespace ccl
