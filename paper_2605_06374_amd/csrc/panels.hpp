// What the kernels with one wave a SIMD share: matrix instructions by register class, LDS tiles as panels.
#ifndef VARLEN_ATTN_PANELS_HPP_
#define VARLEN_ATTN_PANELS_HPP_

#include "tiles.hpp"
#include "staging.hpp"

namespace {

// Scores and their gradients: accumulators in vector registers; nothing touches the results until two further matrix
// instructions have been issued (tiles.hpp). Stationary operand in accumulation registers:
__device__ __forceinline__ void mfma_vgpr_agpr(f32x16& c, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "a"(b));
}
// ... the first of a sum from zero
__device__ __forceinline__ void mfma_vgpr_agpr_first(f32x16& c, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "a"(b));
}
// ... or from an accumulator that stays (statistics of the rows)
__device__ __forceinline__ void mfma_vgpr_agpr_from(f32x16& c, const bf16x8& a, const bf16x8& b, const f32x16& init) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(c) : "v"(a), "a"(b), "v"(init));
}
__device__ __forceinline__ void mfma_vgpr_from(f32x16& c, const bf16x8& a, const bf16x8& b, const f32x16& init) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(c) : "v"(a), "v"(b), "v"(init));
}
template <int KK>
__device__ __forceinline__ void pin_frags_acc(bf16x8 (&f)[KK]) {
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) asm volatile("" : "+a"(f[kk]));
}

// This lane's number, formed anew where it is asked for: what is kept in a register across the units of a workgroup is spilled
__device__ __forceinline__ int fresh_lane() {
  int lane;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
  __builtin_assume(lane >= 0 && lane < 64);
  return lane;
}
// All of an accumulator 0 by one instruction (16 accumulators register by register are 2 KB of code that a unit executes once)
__device__ __forceinline__ void acc_zero(f32x16& acc, const bf16x8& zeros) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %1, 0" : "=a"(acc) : "v"(zeros));
}
__device__ __forceinline__ bf16x8 zero_frag() {
  unsigned x;
  asm volatile("v_mov_b32 %0, 0" : "=v"(x));
  bf16x8 z = __builtin_bit_cast(bf16x8, uint4{x, x, x, x});
  asm volatile("s_nop 1" : "+v"(z));   // (two wait states in front of the matrix instruction)
  return z;
}

// The streamed tiles lie in LDS as panels of 32 columns, [D / 32][64 rows][64 bytes], 16-byte chunk x of row r at x ^ ((r >> 2) & 3):
// 16 neighbouring rows of a chunk, and 4 neighbouring rows of a panel, are 256 bytes that differ in their banks, and every fragment is one
// of four offsets of the lane and a constant (row-major tiles with the swizzle over a whole row take 16 offsets, which this kernel has
// no registers for).
template <int D>
struct PanelOffsets {
  static constexpr int kPanel = kStep * 64;
  int row[2], trans[2];
  __device__ __forceinline__ void init(int lane, int half) {   // `half`: of a stage's rows
    const int h = lane >> 5, c = lane & 31, i = lane & 15, b16 = (lane >> 4) & 1;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      row[x] = (32 * half + c) * 64 + (((2 * x + h) ^ (c >> 2)) & 3) * 16;
      const int r = 4 * h + (i >> 2) + 8 * x;
      trans[x] = (32 * half + r) * 64 + (((2 * b16 + ((i & 3) >> 1)) ^ (r >> 2)) & 3) * 16 + (i & 1) * 8;
    }
  }
  __device__ __forceinline__ void flip() {   // to the other stage
#pragma unroll
    for (int x = 0; x < 2; ++x) { row[x] ^= 2 * kStep * D * 2; trans[x] ^= 2 * kStep * D * 2; }
  }
  // columns 16 kk .. of row c
  __device__ __forceinline__ bf16x8 row_frag(const char* tile, int kk) const { return lds_read_frag(tile, row[kk & 1] + (kk >> 1) * kPanel); }
  // transposed: rows 16 cc + {4h .., 8 + 4h ..}, columns 32 db ..
  __device__ __forceinline__ bf16x8 trans_frag(const char* tile, int cc, int db) const {
    return lds_read_tr8(tile + trans[0] + db * kPanel + cc * 1024, tile + trans[1] + db * kPanel + cc * 1024);
  }
};

}  // namespace

#endif  // VARLEN_ATTN_PANELS_HPP_
