// LDS tiles of the bf16 scan kernels: row-major operand tiles read both as
// MFMA row fragments and, through the transposing LDS read, as column
// fragments, so one copy of an operand serves products over either index.
#pragma once

#include "pdn_device.hpp"

namespace pdn {

typedef __attribute__((address_space(3))) char lds_char;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) floatx4 lds_floatx4;
typedef __attribute__((address_space(3))) float lds_float;

// Byte offset of 16-byte chunk `ch` of row `row` in a tile of NCH chunks a
// row (unpadded).  The chunk is XOR-permuted by row bits 0, 1, 3 and 4: the
// 16 rows of a fragment read (8 (l >> 2) + (l & 3) and four further down)
// fall on distinct 16-byte bank groups, and so do the rows and column groups
// that half a wave of a transposing read touches.  Row bits 2 and 5 do not
// enter, so those steps are constant offsets.
template <int NCH>
__device__ __forceinline__ constexpr int tile_off(int row, int ch) {
  static_assert(NCH == 4 || NCH == 8 || NCH == 16, "tile of 32, 64 or 128 columns");
  constexpr int SH = NCH == 16 ? 0 : NCH == 8 ? 1 : 2;
  const int f = ((((row & 3) >> SH) << 2) | ((row >> 3) & 3)) & (NCH - 1);
  return (row * NCH + (ch ^ f)) * 16;
}

__device__ __forceinline__ bf16x8 lds_frag(const lds_char* p) {
  return *reinterpret_cast<const lds_bf16x8*>(p);
}
__device__ __forceinline__ void lds_put(lds_char* p, bf16x8 v) { *reinterpret_cast<lds_bf16x8*>(p) = v; }
__device__ __forceinline__ void lds_put(lds_char* p, floatx4 v) { *reinterpret_cast<lds_floatx4*>(p) = v; }
__device__ __forceinline__ floatx4 lds_f4(const lds_char* p) { return *reinterpret_cast<const lds_floatx4*>(p); }

// Two transposing reads: within each group of 16 lanes, lane 4 r + q gives
// the address of four adjacent elements (columns 4 q .. 4 q + 3) of row r,
// and lane m receives column m of rows 0 .. 3.  The second read (rows 4 .. 7
// at `second` bytes further) completes the eight contraction elements of an
// MFMA fragment.
__device__ __forceinline__ bf16x8 lds_frag_t(const lds_char* p, int second) {
  lds_s16x4* lo = reinterpret_cast<lds_s16x4*>(const_cast<lds_char*>(p));
  lds_s16x4* hi = reinterpret_cast<lds_s16x4*>(const_cast<lds_char*>(p + second));
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lo);
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16(hi);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

__device__ __forceinline__ floatx4 mfma(bf16x8 a, bf16x8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// two accumulator tiles (rows 4g + i of each) -> the eight contraction
// elements of a fragment
__device__ __forceinline__ bf16x8 pack8(floatx4 lo, floatx4 hi) {
  bf16x8 f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[i] = static_cast<bf16>(lo[i]);
    f[4 + i] = static_cast<bf16>(hi[i]);
  }
  return f;
}

// Workgroup barrier that orders LDS only: outstanding global loads and
// stores stay in flight.
__device__ __forceinline__ void lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// 16-byte store through a raw buffer resource: offsets at or past its byte
// range are dropped by the hardware's range check (no branch).
__device__ __forceinline__ void buf_put16(__amdgpu_buffer_rsrc_t r, uint32_t off, bf16x8 v) {
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, static_cast<int>(off), 0, 0);
}

// Rows [rows][32 columns] of a workspace tensor from a fragment-major LDS
// copy of its transpose: src holds, per column half w (columns 8 (m >> 2) +
// 4 w + (m & 3), m = lane & 15) and 32-row block f, the lanes' 16 bytes (rows
// 32 f + 8 g .. + 7).  Two transposing reads give lane (m, g) columns 8 g ..
// 8 g + 7 of row 32 f + 8 (m >> 2) + 4 hh + (m & 3).
template <int NF>
__device__ __forceinline__ bf16x8 frag_major_row(const lds_char* src, int f, int hh, int l) {
  const int m = l & 15, g = l >> 4;
  const int off = f * 1024 + ((4 * g + (m >> 2)) + 16 * (m & 3)) * 16 + hh * 8;
  return lds_frag_t(src + off, NF * 1024);
}

// ---- the scans' workgroups
constexpr int kCols = 32;      // value columns per workgroup
// Waves: two chain waves, an output wave per 16 rows of a chunk and two
// loaders.  Waves go to the four SIMDs in turn, so the order chain 0, chain 1,
// output 0, 1, loader 0, 1, output 2, 3 puts a loader, which issues little,
// beside each chain wave.
constexpr int kLoaders = 2;
constexpr int scan_threads(int C) { return 64 * (2 + kLoaders + C / 16); }
// The grid of a scan over BH heads, nrole workgroups each, heads in groups of
// eight (one per XCD).  A dimension of a launch holds fewer than 2^32 work
// items, which workgroups of 512 reach at two million heads, so the grid has
// rows of at most kRowHeads heads.  (A split scan's many roles only go with
// few heads.)
constexpr int kRowHeads = 1 << 18;
inline dim3 scan_grid(int64_t BH, int nrole) {
  const int64_t heads = (BH + 7) / 8 * 8;
  return dim3(static_cast<unsigned>((heads < kRowHeads ? heads : kRowHeads) * nrole),
              static_cast<unsigned>((heads + kRowHeads - 1) / kRowHeads));
}
// the workgroup's head and, of the nrole, its role
__device__ __forceinline__ int64_t scan_head(int nrole, int* role) {
  const uint32_t j8 = blockIdx.x >> 3;
  *role = static_cast<int>(j8 % static_cast<uint32_t>(nrole));
  // (BH is below 2^31, so this fits 32 bits, and said so the divisions by H are short)
  return static_cast<uint32_t>(blockIdx.y * kRowHeads + (j8 / static_cast<uint32_t>(nrole)) * 8 + (blockIdx.x & 7));
}
struct RunCtx {
  int64_t b, h, bh;
  int v0;        // first value column
  int c0, c1;    // chunks [c0, c1)
  bool probe;    // a transition run: values (or upstream gradients) are zero
};

// chunk rows as a raw buffer (0 bytes: reads are zeros and cost no traffic)
// (base and size are the same in every lane; said outright, or a descriptor
// the compiler cannot prove uniform costs a loop over its distinct values)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const char* base, uint32_t bytes) {
  const uint64_t p = reinterpret_cast<uint64_t>(base);
  const uint64_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(p)));
  const uint64_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(p >> 32)));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(hi << 32 | lo), 0,
                                           __builtin_amdgcn_readfirstlane(static_cast<int>(bytes)), kBufWord3);
}

// Memory to LDS, 1 KB (64 lanes of 16 bytes) an instruction: unit u of a tile
// of NCH chunks a row is its 64 / NCH rows from u * 64 / NCH.  The XOR order
// of the tile is in the lanes' source offsets.  rows: see row_off (workspace
// rows, which no stride separates, need no limit).
template <int NCH>
__device__ __forceinline__ uint32_t unit_src(int u, int l, uint32_t row_bytes, int rows = 1 << 30) {
  const int r = u * (64 / NCH) + l / NCH;
  const int ch = (tile_off<NCH>(r, l % NCH) / 16) % NCH;   // the chunk at position l % NCH of its row
  return row_off(r, row_bytes, 16u * ch, rows);
}
__device__ __forceinline__ void unit_copy(__amdgpu_buffer_rsrc_t r, uint32_t off, lds_char* dst) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, static_cast<int>(off),
                                           0, 0, 0);
}

// The chunk's per-row scalars (0: lam, 1: w, 2: beta, 3: G) ride in the block of M
// right of the diagonal, which is zero (rows 0 .. C/2 - 1, columns C/2 ..):
// offset in the M tile of the four values of rows 4 q .. 4 q + 3.
template <int C>
__device__ __forceinline__ int scal_off(int x, int q) {
  constexpr int GPR = C / 16;   // groups of four per tile row
  return tile_off<C / 8>(4 * x + q / GPR, C / 16 + q % GPR);
}

// Keeps the LDS reads written before it ahead of what follows: a product's
// fragments are read as a block into registers, one product ahead of use.
// (Left alone the compiler reads each fragment into the same registers right
// before its MFMA and waits out the LDS latency every time.)
__device__ __forceinline__ void reads_done() { asm volatile("" ::: "memory"); }

// Waits until at most N of this wave's memory operations are outstanding
// (they complete in issue order).
template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

}  // namespace pdn
