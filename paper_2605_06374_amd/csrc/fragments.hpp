// Fragment layout of fp32 partial results and bf16 row stores.
#ifndef VARLEN_ATTN_FRAGMENTS_HPP_
#define VARLEN_ATTN_FRAGMENTS_HPP_

#include "tiles.hpp"

namespace {

// ----------------------------------------------------------------------------------------
// Partial results of a cut chain are kept in "fragment layout": the accumulator registers
// exactly as the producing wave holds them, so that every store and load is a contiguous
// 1 KiB per wave: float index (((wave * DB + db) * 4 + rq) * 64 + lane) * 4 + e  for
// accumulator register r = 4 rq + e of column block db.  128 * D floats per tensor.
// ----------------------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void store_frag(float* base, const f32x16 (&acc)[D / 32], int wave,
                                           int lane) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) {
      f32x4 t = {acc[db][4 * rq], acc[db][4 * rq + 1], acc[db][4 * rq + 2], acc[db][4 * rq + 3]};
      *reinterpret_cast<f32x4*>(base + ((((size_t)wave * (D / 32) + db) * 4 + rq) * 64 + lane) * 4) = t;
    }
}
template <int D> constexpr size_t frag_floats() { return (size_t)kTile * D; }
// forward partial: O fragment, then the reference m[4][64] and row sum l[4][64]
template <int D> constexpr size_t fwd_partial_floats() { return frag_floats<D>() + 2 * kThreads; }

// ----------------------------------------------------------------------------------------
// Output rows go through LDS: in an accumulator a lane owns 4 neighbouring columns of its row, so
// that a store straight from it would touch 32 rows with 16 bytes each (512 small writes for a
// wave's 32 rows of 128 columns, where 8 stores of whole rows do): step at 8192 tokens 118.3 -> 113.9
// us (dK/dV 46.6 -> 44.2), 9999 tokens uncut 192.9 -> 185.4 (dK/dV 79.0 -> 73.1), 32768 tokens in
// documents of ordinary length 460.5 -> 445.9.  A tile [32 rows][D] of bf16, with
// the 8-byte slots of a row permuted to spread both sides over the banks: 16-byte chunk `chunk` of row
// r lies at chunk ^ key(r), its halves exchanged in rows 16 .. 31.  (SQ_LDS_BANK_CONFLICT is not zero: 2.4e5
// clocks over all workgroups of a dK/dV launch at 8192 tokens, under 200 of a wave's 100000.)
// ----------------------------------------------------------------------------------------
typedef unsigned u32x2 __attribute__((ext_vector_type(2), may_alias));
typedef unsigned u32x4 __attribute__((ext_vector_type(4), may_alias));
template <int D>
struct RowTile {
  static constexpr int kBytes = 32 * D * 2;
  static constexpr int kChunks = D / 8;   // 16-byte chunks of a row
  static __device__ __forceinline__ int offset(int row, int chunk) {
    const int key = D == 128 ? row & 15 : (row >> 1) & 7;
    return row * (D * 2) + (chunk ^ key) * 16;
  }
  // columns 8 chunk + 4 h .. + 3 of row c
  static __device__ __forceinline__ void put(char* tile, int c, int h, int chunk, uint2 v) {
    *reinterpret_cast<u32x2*>(tile + offset(c, chunk) + (h ^ (c >> 4)) * 8) = u32x2{v.x, v.y};
  }
  static __device__ __forceinline__ uint4 get(const char* tile, int row, int chunk) {
    const u32x4 w = *reinterpret_cast<const u32x4*>(tile + offset(row, chunk));
    return row & 16 ? uint4{w[2], w[3], w[0], w[1]} : uint4{w[0], w[1], w[2], w[3]};
  }
};
// A wave's 32 accumulator rows as bf16 at `out` (its first row), of which `rows` exist.  `tile`:
// kBytes of LDS that no other wave uses now.
template <int D>
__device__ __forceinline__ void store_rows(char* tile, __bf16* out, size_t row_stride, int rows,
                                           const f32x16 (&acc)[D / 32], int lane, float mul) {
  using T = RowTile<D>;
  const int h = lane >> 5, c = lane & 31;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int rq = 0; rq < 4; ++rq)
      T::put(tile, c, h, 4 * db + rq,
             pack4(acc[db][4 * rq] * mul, acc[db][4 * rq + 1] * mul, acc[db][4 * rq + 2] * mul, acc[db][4 * rq + 3] * mul));
  asm volatile("" ::: "memory");   // the LDS serves a wave's accesses in order
  constexpr int kRows = 64 / T::kChunks;   // per store
  const int chunk = lane % T::kChunks;
#pragma unroll
  for (int j = 0; j < 32 / kRows; ++j) {
    const int row = kRows * j + lane / T::kChunks;
    const uint4 w = T::get(tile, row, chunk);
    if (row < rows) *reinterpret_cast<uint4*>(out + row * row_stride + 8 * chunk) = w;
  }
}

}  // namespace

#endif  // VARLEN_ATTN_FRAGMENTS_HPP_
