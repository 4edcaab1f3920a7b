// Vector types, constants, MFMA wrapper and swizzled LDS tile addressing shared by every kernel.
//
// Register/lane conventions used by every kernel (L = lane, h = L / 32, c = L % 32):
//   MFMA 32x32x16:  A[i][k]: lane holds i = c, k = 8h + e (e = 0..7)
//                   B[k][j]: lane holds j = c, k = 8h + e
//                   C[i][j]: lane holds j = c, i = 8 (r / 4) + 4h + r % 4 (r = 0..15)
// The kernels always put the softmax row index on the lane (j = c) so that row statistics
// are per-lane scalars, and feed the exponentiated scores straight back as a B operand:
// registers 8cc..8cc+7 of a C tile are the k positions of the cc-th 16-deep slice, standing
// for rows 16cc + 4h + {0..3} and 16cc + 8 + 4h + {0..3}.  The matching A operand is a
// transposed read of a row-major LDS tile (ds_read_b64_tr_b16, twice).
#ifndef VARLEN_ATTN_TILES_HPP_
#define VARLEN_ATTN_TILES_HPP_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "varlen_attn.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kTile = VARLEN_ATTN_TILE_ROWS;  // rows of a work item (4 waves x 32)
constexpr int kStep = VARLEN_ATTN_STEP_ROWS;  // rows staged per iteration of a chain
constexpr int kThreads = 256;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
// The forward renews the reference of its exponentials when the row sum of a sub-step exceeds 2^8, and
// puts it 12 powers of two above the row's maximum.  The sum bounds P, and with it how far the
// unnormalised O lies above O: with 2^24 in its place values |V| of 2^112 overflowed.  The room below
// makes renewals rare where scores keep growing (forward at 32768 tokens in 11 documents, scores with
// a standard deviation of 9, against a bound of 2^24: 1.13 times as long without the room, 1.02 with it;
// the same up to a standard deviation of 2).
constexpr float kRefSumMax = 256.f, kRefRoom = 12.f;

// dK / dV: the matrix instructions of S start from -LSE / scale, which overflows for scales below LSE / 2^128.
// Below 2^-120 the K fragments of S are therefore multiplied by 2^-32 and the scale that S and -LSE are
// counted in is 2^32 times larger; what K loses at the bottom of its range is below 2^-86 of a score.
__device__ __forceinline__ float score_fold(float scale) { return scale < 0x1p-120f ? 0x1p-32f : 1.0f; }
__device__ __forceinline__ float folded_scale(float scale) { return scale < 0x1p-120f ? scale * 0x1p32f : scale; }

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>): a loop whose body may hold
// scheduling fences (an ordinary loop that holds one is not unrolled).
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// ----------------------------------------------------------------------------------------
// LDS tiles: row-major [rows][D] bf16, addressed in 16-byte chunks with an XOR swizzle that
// keeps both the row-fragment reads (ds_read_b128, 32 rows x one chunk) and the transposed
// reads (ds_read_b64_tr_b16, 4 rows x 64 bytes per half-wave) spread over the banks.
// ----------------------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ int swz(int row) {
  if constexpr (D == 128) return ((row & 3) << 2) | ((row >> 2) & 3);
  else return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
}
template <int D>
__device__ __forceinline__ int chunk_off(int row, int chunk) {  // in bytes
  return (row * (D / 8) + (chunk ^ swz<D>(row))) * 16;
}

__device__ __forceinline__ bf16x8 lds_read_frag(const char* tile, int byte_off) {
  return *reinterpret_cast<const bf16x8*>(tile + byte_off);
}

// Transposed 4x(16 lanes) read: lane i of each 16-lane group passes the address of 4
// consecutive columns of row (i / 4); it receives rows 0..3 at column i of the group.
__device__ __forceinline__ bf16x4 lds_read_tr(const char* p) {
  s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (s16x4 __attribute__((address_space(3)))*)(p));
  return __builtin_bit_cast(bf16x4, v);
}

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// The same with the accumulator kept in vector registers whatever the compiler would choose.  The
// compiler's wait states cover neither its operands nor its result: whoever uses it keeps the distance,
// by mfma_vgpr_settle() (short.hpp) or by two further matrix instructions behind a fence (dK/dV), and
// tests/test_wait_states.py checks the distances on the compiled code.
__device__ __forceinline__ void mfma_vgpr(f32x16& c, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}

// ... and the first of a sum starts from zero: its accumulator is not written by vector instructions
// right in front of it (a hazard that the compiler does not see either).
template <bool FIRST>
__device__ __forceinline__ void mfma_vgpr_acc(f32x16& c, const bf16x8& a, const bf16x8& b) {
  if constexpr (FIRST) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
  else mfma_vgpr(c, a, b);
}
// Between the last mfma_vgpr of an accumulator and the first vector instruction that reads it: 16
// wait states (an 8-pass matrix instruction needs 12), fenced on both sides.
__device__ __forceinline__ void mfma_vgpr_settle() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 15");
  __builtin_amdgcn_sched_barrier(0);
}

// value held by the same column in the other half of the wave (lane ^ 32), combined by op
__device__ __forceinline__ float half_max(float x) {
  unsigned u = __builtin_bit_cast(unsigned, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __builtin_fmaxf(__builtin_bit_cast(float, (unsigned)r[0]),
                         __builtin_bit_cast(float, (unsigned)r[1]));
}
__device__ __forceinline__ float half_sum(float x) {
  unsigned u = __builtin_bit_cast(unsigned, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}

// acc + a . b, pairs of products added in fp32
__device__ __forceinline__ float dot8(const bf16x8& a, const bf16x8& b, float acc) {
#pragma unroll
  for (int e = 0; e < 8; e += 2)
    acc = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{a[e], a[e + 1]}, bf16x2{b[e], b[e + 1]}, acc, false);
  return acc;
}

__device__ __forceinline__ bf16x8 pack8(const f32x16& v, int first) {
  bf16x8 out;
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    f32x2 t = {v[first + e], v[first + e + 1]};
    bf16x2 b = __builtin_convertvector(t, bf16x2);
    out[e] = b[0];
    out[e + 1] = b[1];
  }
  return out;
}

// registers 4 rq .. 4 rq + 3 of an accumulator
__device__ __forceinline__ void set4(f32x16& v, int rq, f32x4 x) {
#pragma unroll
  for (int e = 0; e < 4; ++e) v[4 * rq + e] = x[e];
}

__device__ __forceinline__ uint2 pack4(float a, float b, float c, float d) {
  f32x2 t0 = {a, b}, t1 = {c, d};
  bf16x2 b0 = __builtin_convertvector(t0, bf16x2), b1 = __builtin_convertvector(t1, bf16x2);
  return uint2{__builtin_bit_cast(unsigned, b0), __builtin_bit_cast(unsigned, b1)};
}

}  // namespace

#endif  // VARLEN_ATTN_TILES_HPP_
