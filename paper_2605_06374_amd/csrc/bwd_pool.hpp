// Backward as one pool of work: dQ units and dK/dV units drawn by resident workgroups.
#ifndef VARLEN_ATTN_BWD_POOL_HPP_
#define VARLEN_ATTN_BWD_POOL_HPP_

#include "tiles.hpp"
#include "staging.hpp"
#include "panels.hpp"
#include "fragments.hpp"
#include "plan.hpp"

namespace {

// ----------------------------------------------------------------------------------------
// Backward (the rule: pooled_backward() in varlen_attn.hip; figures without a head size are for 128).  One workgroup per
// compute unit stays and draws units, column units (dK, dV) first, then units of dQ, longest first within each: the short dQ
// units fill what the column units leave idle, where a kernel each has a tail, a burst of first loads and a launch of its own.
// dQ has units of its own (plan.hpp): in the pool a chain needs no cut until it would outlast the rest, which leaves a quarter
// of the partial results at 8192 tokens.  Nothing depends on the order in which units are drawn, so that the results are
// reproducible.  The price is D: both kinds need it, so it comes from a pass in front (bwd_prep_kernel).
//
// What bounds it: at 512 registers one wave per SIMD issues everything, and on large microbatches the clock, which the power
// limit takes down to 1.7 - 2.0 GHz on real operands (2.2 on zeros).  A wave owns 64 of a unit's 128 rows against half of the
// 64 streamed rows of every stage, so that a fragment from LDS feeds two matrix instructions; with 32 rows a wave against all
// of the stage the LDS was busy for 0.9 of the matrix pipe's time.  A stage of 64 rows, one wave's 32 rows before / now, 8192
// tokens in 9 documents: columns 1.61 / 1.43 us, dQ 1.23 / 1.12; 32768 tokens in 11 documents 1.80 / 1.65, 1.33 / 1.25.  The
// matrix instructions alone (no vector work, LDS reads or loads) take 1.18, 0.89, 1.36 and 0.99.  The price is paid between two
// sweeps: the halves of a stage meet in LDS, which the next unit's rows are landing in as well (LDS writes run at 77 bytes a
// clock, reads at 170): a column unit's results take 3.3 us there instead of 1.8, which short documents pay for: backward of 56
// packs of documents of 60 to 180 tokens 0.94 to 1.19, 1.00 in the mean, times as fast as with 32 rows a wave (up to 32 tokens
// are spared it: lower_half_only(); 22 packs 1.00 to 1.30).  Whole steps: 8192 tokens 108.9 -> 106.1 us, 7001 80.8 -> 77.5,
// 16384 with 8 q heads on one kv head 626 -> 601, 32768 in 35 documents 426 -> 409, in 11 1683 -> 1604, 131072 in one 32.3 ->
// 30.6 ms.
//
// Both sweeps are pipelined by hand; vector work and LDS reads ride on matrix instructions, the next stage's loads on those of S:
//   columns  S(0, 1) | dP(0, 1) with P | dV(0, 1) with P, dS | dK(0, 1) with dS | wait, barrier |
//            the last of dK with the next stage's first reads
//   dQ       S(0) | S(1) with P(0) | dP(0) with P(0), P(1) | dP(1) with P(1), dS(0) | dQ(0) with dS(1) |
//            wait, barrier | dQ(1) with the next reads
// (0, 1: the wave's two blocks of 32 stationary rows).  The operands of what follows a barrier are in registers by then, so
// that no wave meets an empty matrix pipe behind it.  The sums of a column unit take all 256 accumulation registers and its
// stationary fragments half of the vector registers; dQ's sums and stationary fragments share the accumulation registers.
// Measured and left out: row units first, which publish D themselves, with a wait in front of the column units (loads past the
// L2 and 250 increments of one counter: 44 instead of 23 us at 4096 tokens); the next unit's stationary tiles through LDS while
// the last stages run (its bookkeeping costs each of those stages as much as the loads would); stages unrolled in pairs (a
// third more code, no faster); output rows stored from registers, 32 bytes of a row at a time (a step at 32768 tokens in 35
// documents 409 -> 420 us).
// ----------------------------------------------------------------------------------------

// A wave-uniform condition as a vector value: the branch is then by the execution mask, the two forms of a stage lie one behind
// the other and the accumulators keep their registers (a scalar branch copies them).
__device__ __forceinline__ bool by_exec_mask(bool x) {
  int v = x;
  asm volatile("" : "+v"(v));
  return v != 0;
}
// x / d for a divisor that stays the same, wave-uniform
struct Divisor {
  unsigned d, m;   // m = floor(2^32 / d), or less by one: the quotient misses by at most one
  __device__ __forceinline__ void init(int d_) {
    d = (unsigned)d_;
    m = 0xFFFFFFFFu / d;
  }
  __device__ __forceinline__ int operator()(int x) const {
    const unsigned q = __umulhi((unsigned)x, m);
    return (int)(q + ((unsigned)x - q * d >= d ? 1 : 0));
  }
};

// The units of a pool are dealt by tickets, column units first, one counter per group of heads (the heads whose K, V, Q
// and dO lines share the L2 of the group's XCDs).  A workgroup's first ticket is its own number in its group, later
// ones come from the counter.
struct TicketGroup {
  int index, stride, members, first;   // counter; head groups per unit number; workgroups of the group; own number
  int n_col, total;
  Divisor heads, hpu, per;
  __device__ __forceinline__ void init(int bid, int groups, int Hq, int hpu_) {
    const int Hv = Hq / hpu_, xcd = bid % 8;
    int heads_;
    if (8 % Hv == 0) { index = xcd % Hv; heads_ = 1; first = (bid / 8) * (8 / Hv) + xcd / Hv; members = groups / Hv; }
    else if (Hv % 8 == 0) { index = xcd; heads_ = Hv / 8; first = bid / 8; members = groups / 8; }
    else { index = 0; heads_ = Hv; first = bid; members = groups; }
    stride = Hv % 8 == 0 ? 8 : 1;
    heads.init(heads_);
    hpu.init(hpu_);
    per.init(heads_ * hpu_);
  }
  __device__ __forceinline__ void set(int col_units, int dq_units) {
    n_col = col_units * (int)heads.d;
    total = n_col + dq_units * (int)per.d;
  }
  __device__ __forceinline__ void decode(int t, int& unit, int& head) const {
    if (t < n_col) {
      unit = heads(t);
      head = (index + stride * (t - unit * (int)heads.d)) * (int)hpu.d;
    } else {
      const int r = t - n_col;
      unit = per(r);
      const int j = r - unit * (int)per.d, v = hpu(j);
      head = (index + stride * v) * (int)hpu.d + (j - v * (int)hpu.d);
    }
  }
};

// The next ticket: thread 0 asks for it in front of a unit's last stage but one and passes it on through LDS in front of
// the last, whose barrier publishes it.  (Units of one stage: when the unit is opened; the answer takes about as long as a stage.)
struct Tickets {
  int* counter;
  int* lds;
  int next;
  __device__ __forceinline__ void step(int pass) {
    if (threadIdx.x == 0) {
      if (pass) *lds = next;
      else next = atomicAdd(counter, 1);
    }
    __builtin_amdgcn_wave_barrier();   // (the branch ends here, so that what follows stays wave-uniform)
  }
  __device__ __forceinline__ int take() const {
    const int t = __builtin_amdgcn_readfirstlane(*lds);
    __syncthreads();   // (the last stage's read-ahead ends; results meet where the ticket was)
    return t;
  }
};

template <int D>
struct BwdArgs {
  const __bf16 *q, *k, *v, *d_o;
  const float *neg_lse, *neg_dsum;
  const varlen_attn_plan_header* hdr;
  const varlen_attn_unit *col_units, *dq_units, *row_units;
  __bf16 *dq, *dk, *dv;
  float *col_partials, *row_partials;
  int N, Hq, Hkv, max_units;
  float scale;
  int* tickets;
};

// LDS of a workgroup, all there is: two stages of two streamed tiles (K and V, or Q and dO), next to each other; the 128 rows
// of the two stationary tiles on their way to registers; the statistics of the streamed queries (-LSE / scale [64], -D [64] per
// stage, two copies, one per pair of waves).  Between two sweeps results meet in the second stage's half and behind the
// stationary tiles, 16 KB a wave, while the next unit's first stage and stationary rows are landing.
template <int D>
struct BwdLds {
  static constexpr int kHalf = kStep * D * 2, kStage = 2 * kHalf, kStat = 512, kFixed = kTile * D * 2, kMeet = 32 * D * 4;
  static constexpr int kFixeds = 2 * kStage, kStats = kFixeds + 2 * kFixed, kTicket = kStats + 4 * kStat;
  static __device__ __forceinline__ int meet(int wave) { return (wave & 2 ? kStats : kStage) + (wave & 1) * kMeet; }
  // 64 columns of 32 output rows, in the second stage's half: 16-byte chunk x of row r at x * kOutChunk + 16 r, spread over the
  // banks both ways
  static constexpr int kOutChunk = 32 * 16 + 32, kOut = 8 * kOutChunk, kOuts = 4 * kOut <= kStage ? kStage : kStats + 2 * kMeet;
  static constexpr int kBytes = 4 * kOut <= kStage ? kStats + 2 * kMeet : kOuts + 4 * kOut;
};
static_assert(BwdLds<128>::kBytes == 160 * 1024, "of a compute unit");

// Accumulator number I of a kernel that keeps its sums in accumulation registers 16 I .. 16 I + 15, by inline assembly: its
// values in vector registers, or in LDS (four pieces of 1 KB a wave, from `OFFSET` on).  An element that the compiler takes out
// itself draws the whole accumulator into vector registers, and all of them right behind the sweep, where they are spilled.
#define VARLEN_ATTN_ACCUMULATORS(X)                                                                                       \
  X(0, "0:15", "0:3", "4:7", "8:11", "12:15", 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15)                        \
  X(1, "16:31", "16:19", "20:23", "24:27", "28:31", 16, 17, 18, 19, 20, 21, 22, 23, 24, 25, 26, 27, 28, 29, 30, 31) \
  X(2, "32:47", "32:35", "36:39", "40:43", "44:47", 32, 33, 34, 35, 36, 37, 38, 39, 40, 41, 42, 43, 44, 45, 46, 47) \
  X(3, "48:63", "48:51", "52:55", "56:59", "60:63", 48, 49, 50, 51, 52, 53, 54, 55, 56, 57, 58, 59, 60, 61, 62, 63) \
  X(4, "64:79", "64:67", "68:71", "72:75", "76:79", 64, 65, 66, 67, 68, 69, 70, 71, 72, 73, 74, 75, 76, 77, 78, 79) \
  X(5, "80:95", "80:83", "84:87", "88:91", "92:95", 80, 81, 82, 83, 84, 85, 86, 87, 88, 89, 90, 91, 92, 93, 94, 95) \
  X(6, "96:111", "96:99", "100:103", "104:107", "108:111", 96, 97, 98, 99, 100, 101, 102, 103, 104, 105, 106, 107, 108, 109, 110, 111) \
  X(7, "112:127", "112:115", "116:119", "120:123", "124:127", 112, 113, 114, 115, 116, 117, 118, 119, 120, 121, 122, 123, 124, 125, 126, 127) \
  X(8, "128:143", "128:131", "132:135", "136:139", "140:143", 128, 129, 130, 131, 132, 133, 134, 135, 136, 137, 138, 139, 140, 141, 142, 143) \
  X(9, "144:159", "144:147", "148:151", "152:155", "156:159", 144, 145, 146, 147, 148, 149, 150, 151, 152, 153, 154, 155, 156, 157, 158, 159) \
  X(10, "160:175", "160:163", "164:167", "168:171", "172:175", 160, 161, 162, 163, 164, 165, 166, 167, 168, 169, 170, 171, 172, 173, 174, 175) \
  X(11, "176:191", "176:179", "180:183", "184:187", "188:191", 176, 177, 178, 179, 180, 181, 182, 183, 184, 185, 186, 187, 188, 189, 190, 191) \
  X(12, "192:207", "192:195", "196:199", "200:203", "204:207", 192, 193, 194, 195, 196, 197, 198, 199, 200, 201, 202, 203, 204, 205, 206, 207) \
  X(13, "208:223", "208:211", "212:215", "216:219", "220:223", 208, 209, 210, 211, 212, 213, 214, 215, 216, 217, 218, 219, 220, 221, 222, 223) \
  X(14, "224:239", "224:227", "228:231", "232:235", "236:239", 224, 225, 226, 227, 228, 229, 230, 231, 232, 233, 234, 235, 236, 237, 238, 239) \
  X(15, "240:255", "240:243", "244:247", "248:251", "252:255", 240, 241, 242, 243, 244, 245, 246, 247, 248, 249, 250, 251, 252, 253, 254, 255)
template <int I>
__device__ __forceinline__ void acc_values(const f32x16& acc, float (&x)[16]) {
#define VARLEN_ATTN_VALUES(i, all, q0, q1, q2, q3, r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15)                    \
  if constexpr (I == i)                                                                                                                \
    asm volatile("v_accvgpr_read_b32 %0, a" #r0 "\n\tv_accvgpr_read_b32 %1, a" #r1 "\n\tv_accvgpr_read_b32 %2, a" #r2                   \
                 "\n\tv_accvgpr_read_b32 %3, a" #r3 "\n\tv_accvgpr_read_b32 %4, a" #r4 "\n\tv_accvgpr_read_b32 %5, a" #r5               \
                 "\n\tv_accvgpr_read_b32 %6, a" #r6 "\n\tv_accvgpr_read_b32 %7, a" #r7 "\n\tv_accvgpr_read_b32 %8, a" #r8               \
                 "\n\tv_accvgpr_read_b32 %9, a" #r9 "\n\tv_accvgpr_read_b32 %10, a" #r10 "\n\tv_accvgpr_read_b32 %11, a" #r11           \
                 "\n\tv_accvgpr_read_b32 %12, a" #r12 "\n\tv_accvgpr_read_b32 %13, a" #r13 "\n\tv_accvgpr_read_b32 %14, a" #r14         \
                 "\n\tv_accvgpr_read_b32 %15, a" #r15                                                                                  \
                 : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]), "=&v"(x[6]), "=&v"(x[7]), "=&v"(x[8]), \
                   "=&v"(x[9]), "=&v"(x[10]), "=&v"(x[11]), "=&v"(x[12]), "=&v"(x[13]), "=&v"(x[14]), "=&v"(x[15])                      \
                 : "{a[" all "]}"(acc));
  VARLEN_ATTN_ACCUMULATORS(VARLEN_ATTN_VALUES)
#undef VARLEN_ATTN_VALUES
}
template <int I, int OFFSET>
__device__ __forceinline__ void acc_to_lds(const f32x16& acc, unsigned lds_addr) {
#define VARLEN_ATTN_WRITE(i, all, q0, q1, q2, q3, r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15)                  \
  if constexpr (I == i)                                                                                                             \
    asm volatile("ds_write_b128 %0, a[" q0 "] offset:%2\n\tds_write_b128 %0, a[" q1 "] offset:%3"                                    \
                 "\n\tds_write_b128 %0, a[" q2 "] offset:%4\n\tds_write_b128 %0, a[" q3 "] offset:%5"                                    \
                 :                                                                                                                  \
                 : "v"(lds_addr), "{a[" all "]}"(acc), "n"(OFFSET), "n"(OFFSET + 1024), "n"(OFFSET + 2048), "n"(OFFSET + 3072)       \
                 : "memory");
  VARLEN_ATTN_ACCUMULATORS(VARLEN_ATTN_WRITE)
#undef VARLEN_ATTN_WRITE
}

// The two halves of a stage meet: accumulators GIVE .. of this wave go to the wave of the other half (give(), a barrier behind
// it in take()), whose accumulators come back in fragment order, to be added to TAKE ..  All waves; those without a row of the
// tile meet the barriers only.
template <int D, int GIVE>
__device__ __forceinline__ void give(char* smem, int wave, bool any_rows, const f32x16 (&acc)[D / 32]) {
  if (!any_rows) return;
  const unsigned own = lds_addr_of(smem) + BwdLds<D>::meet(wave) + fresh_lane() * 16;
  static_for<D / 32>([&](auto db) __attribute__((always_inline)) { acc_to_lds<GIVE + db, db * 4096>(acc[db], own); });
}
template <int D, int TAKE>
__device__ __forceinline__ void take(char* smem, int wave, int lane, const f32x16 (&acc)[D / 32], f32x4 (&other)[D / 8], float (&mine)[D / 32][16]) {
  const char* const from = smem + BwdLds<D>::meet(wave ^ 2) + lane * 16;
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __syncthreads();
#pragma unroll
  for (int i = 0; i < D / 8; ++i) other[i] = *reinterpret_cast<const f32x4*>(from + i * 1024);
  static_for<D / 32>([&](auto db) __attribute__((always_inline)) { acc_values<TAKE + db>(acc[db], mine[db]); });
  __syncthreads();   // (the share may be overwritten)
}
__device__ __forceinline__ void skip_take() {
  __syncthreads();
  __syncthreads();
}
template <int D>
__device__ __forceinline__ void add(f32x4 (&x)[D / 8], const float (&mine)[D / 32][16]) {
#pragma unroll
  for (int i = 0; i < D / 8; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) x[i][e] += mine[i / 4][4 * (i % 4) + e];
}

// Has this wave a row of the unit's tile?
__device__ __forceinline__ bool has_rows(const varlen_attn_unit& it, int wave) { return it.row0 + 64 * (wave & 1) < it.doc_end; }
// The streamed rows of a unit end in the lower half of its only stage: what wave 0 has is the result, and no halves meet.  Two
// branches a unit of other tiles.  32 rows a wave / meeting always / so, backward, resident buffers: 1250 documents of 32
// tokens 56.8 / 60.2 / 51.9 us, 489 of 8 to 100, 8 heads, 162.9 / 176.1 / 158.8; documents of 60 to 200 tokens 0.987 .. 1.005
// of the speed without it, 32768 tokens in 35 1.005.
__device__ __forceinline__ bool lower_half_only(const varlen_attn_unit& it, bool columns) {
  return it.doc_end - (columns ? it.row0 : it.doc_start) <= kStep / 2;
}
// Block of 32 rows of the unit's tile that this wave stores
__device__ __forceinline__ int own_block(int wave) { return 2 * (wave & 1) + (wave >> 1); }

template <int D>
__device__ __forceinline__ void store_partial(float* partial, int wave, int lane, const f32x4 (&x)[D / 8]) {
  float* const p = partial + ((size_t)own_block(wave) * (D / 8) * 64 + lane) * 4;
#pragma unroll
  for (int i = 0; i < D / 8; ++i) *reinterpret_cast<f32x4*>(p + i * 256) = x[i];
}

// ... of wave 0, whose sums are the results
template <int D>
__device__ __forceinline__ void store_partial(float* partial, const float (&x)[D / 32][16], int lane) {
  float* const p = partial + lane * 4;
#pragma unroll
  for (int i = 0; i < D / 8; ++i)
    *reinterpret_cast<f32x4*>(p + i * 256) = f32x4{x[i / 4][4 * (i % 4)], x[i / 4][4 * (i % 4) + 1], x[i / 4][4 * (i % 4) + 2], x[i / 4][4 * (i % 4) + 3]};
}
template <int D>
__device__ __forceinline__ void pack(uint2 (&w)[D / 8], const float (&x)[D / 32][16], float mul) {
#pragma unroll
  for (int i = 0; i < D / 8; ++i)
    w[i] = pack4(x[i / 4][4 * (i % 4)] * mul, x[i / 4][4 * (i % 4) + 1] * mul, x[i / 4][4 * (i % 4) + 2] * mul, x[i / 4][4 * (i % 4) + 3] * mul);
}

// bf16 rows by way of LDS, 64 columns at a time in runs of 128 bytes; buffer stores, which leave out what lies behind the last row
template <int D>
__device__ __forceinline__ void store_bf16(char* smem, int wave, int lane, const varlen_attn_unit& it, const uint2 (&x)[D / 8], __bf16* out, int heads,
                                           int head) {
  using L = BwdLds<D>;
  const int row0 = it.row0 + 32 * own_block(wave), rows = min(max(it.doc_end - row0, 0), 32);
  char* const tile = smem + L::kOuts + wave * L::kOut;
  char* const put = tile + 16 * (lane & 31) + 8 * (lane >> 5);
  const char* const get = tile + (lane & 7) * L::kOutChunk + (lane >> 3) * 16;
  const unsigned stride = (unsigned)heads * (D * 2), offset = (unsigned)(lane >> 3) * stride + (lane & 7) * 16;
  const __amdgpu_buffer_rsrc_t rsrc =
      __builtin_amdgcn_make_buffer_rsrc((void*)uniform64(out + ((size_t)row0 * heads + head) * D), 0,
                                        __builtin_amdgcn_readfirstlane(rows ? (rows - 1) * stride + D * 2 : 0), 0x00027000);
#pragma unroll
  for (int turn = 0; turn < D / 64; ++turn) {
#pragma unroll
    for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x2*>(put + i * L::kOutChunk) = u32x2{x[8 * turn + i].x, x[8 * turn + i].y};
    asm volatile("" ::: "memory");   // the LDS serves a wave's accesses in order
#pragma unroll
    for (int j = 0; j < 4; ++j)
      __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4*>(get + 128 * j), rsrc, offset + 8 * j * stride + 128 * turn, 0, 0);
    asm volatile("" ::: "memory");
  }
}

// A wave's direct-to-LDS loads of its 16 rows of a stage of two such tiles with a common row stride, one panel a piece
template <int D>
struct PanelStream {
  static constexpr int kPanels = D / 32, kPieces = 2 * kPanels;
  unsigned own, col;               // offset of this lane's 16 bytes from the stage's first row, the column's share of it
  unsigned stride, last;           // (uniform) bytes from row to row, to the last row that exists
  unsigned long long a_next, b_next, stage_stride;
  __device__ __forceinline__ void init(int wave, int lane, unsigned stride_bytes) {
    stride = stride_bytes;
    stage_stride = (unsigned long long)kStep * stride_bytes;
    col = (unsigned)(((lane ^ (lane >> 4)) & 3) * 16);
    own = (unsigned)(16 * wave + (lane >> 2)) * stride + col;
  }
  __device__ __forceinline__ void start(const void* a, const void* b) { a_next = uniform64(a); b_next = uniform64(b); }
  // the next stage starts at row `row0`; rows above row_last are clamped to it
  __device__ __forceinline__ void aim(int row0, int row_last) { last = (unsigned)min(row_last - row0, kStep - 1) * stride; }
  __device__ __forceinline__ void advance() { a_next += stage_stride; b_next += stage_stride; }
  __device__ __forceinline__ unsigned offset() const { return min(own, last + col); }
  // Piece P to this wave's first kilobyte `lds` of the first tile, the second tile behind the first: the destination, and, an
  // instruction later at the earliest, the load.  The load's constant offset counts on both sides, in memory and in LDS.
  template <int P>
  static __device__ __forceinline__ void aim_piece(unsigned lds) {
    constexpr int i = P % kPanels;
    asm volatile("s_add_u32 m0, %0, %1" : : "s"(lds), "n"((P < kPanels ? 0 : kStep * D * 2) + i * (PanelOffsets<D>::kPanel - 64)) : "scc");
  }
  template <int P>
  __device__ __forceinline__ void load_piece(unsigned voff) const {
    asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" : : "v"(voff), "s"(P < kPanels ? a_next : b_next), "n"(64 * (P % kPanels)) : "memory");
  }
  __device__ __forceinline__ void load_stage(unsigned lds) const {
    const unsigned voff = offset();
    static_for<kPieces>([&](auto p) __attribute__((always_inline)) {
      aim_piece<decltype(p)::value>(lds);
      asm volatile("s_nop 0");
      load_piece<decltype(p)::value>(voff);
    });
  }
};

// The 128 rows of a unit's two stationary tiles, with a common row stride, to LDS: panels of 32 columns as above, 128 rows each; then this
// wave's fragments of them to registers.  (Straight to registers every load would touch 32 rows, 64 clocks each of the path to memory.)
template <int D>
struct FixedTiles {
  static constexpr int kPanel = kTile * 64;
  static __device__ __forceinline__ void request(const __bf16* a, const __bf16* b, unsigned stride, int row0, int row_last, char* smem, int wave) {
    const int lane = fresh_lane();
    const unsigned long long a0 = uniform64(a), b0 = uniform64(b);
    const unsigned lds = lds_addr_of(smem) + BwdLds<D>::kFixeds + wave * 2048;
    const unsigned col = (unsigned)(((lane ^ (lane >> 4)) & 3) * 16);
#pragma unroll
    for (int half = 0; half < 2; ++half) {   // 16 rows each
      if (32 * wave + 16 * half > row_last - row0) break;   // (fragments of rows that do not exist may be anything)
      const unsigned voff = (unsigned)min(32 * wave + 16 * half + (lane >> 2), row_last - row0) * stride + col;
#pragma unroll
      for (int db = 0; db < D / 32; ++db) {
        dma16(a0 + 64 * db, voff, lds + half * 1024 + db * kPanel);
        dma16(b0 + 64 * db, voff, lds + half * 1024 + db * kPanel + BwdLds<D>::kFixed);
      }
    }
  }
  // the first tile times `factor` (tiny softmax scales only)
  static __device__ __forceinline__ void fold(char* smem, int wave, float factor) {
    bf16x8* const mine = reinterpret_cast<bf16x8*>(smem + BwdLds<D>::kFixeds) + 64 * wave + fresh_lane();
#pragma unroll 1
    for (int i = 0; i < BwdLds<D>::kFixed / 16; i += kThreads) {
      bf16x8 x = mine[i];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = (__bf16)((float)x[e] * factor);
      mine[i] = x;
    }
    __syncthreads();
  }
  // block 0 is the one whose results this wave will store: rows 32 half .. of its 64
  static __device__ __forceinline__ void read(const char* smem, const PanelOffsets<D>& fo, int wave, bf16x8 (&a)[2][D / 16], bf16x8 (&b)[2][D / 16]) {
    const char* const tile = smem + BwdLds<D>::kFixeds;
    const int half = wave >> 1;
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) {
        const int off = fo.row[kk & 1] + (64 * (wave & 1) + 32 * (blk ^ half) - 32 * half) * 64 + (kk >> 1) * kPanel;
        a[blk][kk] = lds_read_frag(tile, off);
        b[blk][kk] = lds_read_frag(tile, off + BwdLds<D>::kFixed);
      }
  }
};

// The units are objects: open() sends the loads of a unit's first stage and of its stationary rows on their way, sweep()
// walks its chain, store() writes the results.  The next unit is opened before the results of the last one are stored.
// Wave w owns 64 of the 128 stationary rows, those of w & 1, against one half, w >> 1, of the 64 rows of every stage: each fragment
// that comes from LDS feeds two matrix instructions.  Its two blocks of 32 rows are numbered so that it stores block 0.
template <int D>
struct DqUnit {
  static constexpr int KK = D / 16, DB = D / 32, kStage = BwdLds<D>::kStage;
  varlen_attn_unit it;
  int head;
  PanelStream<D> stream;
  float neg_lse_row[2], neg_dsum_row[2];

  __device__ __forceinline__ void open(const BwdArgs<D>& a, const varlen_attn_unit& unit, int head_, int kvh, char* smem, int wave, Tickets& tickets) {
    it = unit;
    head = head_;
    if (it.step_end - it.step_begin == 1) tickets.step(0);
    const int Hq = a.Hq, Hkv = a.Hkv;
    const int lane = fresh_lane();
    const int kv_first = it.doc_start + kStep * it.step_begin;
    stream.init(wave, lane, (unsigned)((size_t)Hkv * D * 2));
    stream.start(a.k + ((size_t)kv_first * Hkv + kvh) * D, a.v + ((size_t)kv_first * Hkv + kvh) * D);
    stream.aim(kv_first, it.doc_end - 1);
    stream.load_stage(lds_addr_of(smem) + wave * 1024);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int row = min(it.row0 + 64 * (wave & 1) + 32 * (b ^ (wave >> 1)) + (lane & 31), it.doc_end - 1);
      neg_lse_row[b] = a.neg_lse[(size_t)head * a.N + row];
      neg_dsum_row[b] = a.neg_dsum[(size_t)head * a.N + row];
    }
    // rows past the document end: duplicates, never stored
    FixedTiles<D>::request(a.q + ((size_t)it.row0 * Hq + head) * D, a.d_o + ((size_t)it.row0 * Hq + head) * D, (unsigned)(Hq * D * 2), it.row0,
                           it.doc_end - 1, smem, wave);
  }

  // S^T = K Q^T, dP^T = V dO^T, dQ^T += K^T dS^T.  `follows`: this wave issued stores of another unit, D / 16 at least, behind
  // this unit's loads (none where it had no rows of that unit).
  template <typename Tickets>
  __device__ __forceinline__ void sweep(const BwdArgs<D>& a, bool follows, char* smem, int wave, f32x16 (&acc)[2][DB], Tickets& tickets) {
    float scale = a.scale;
    asm volatile("" : "+s"(scale));
    const float cs = folded_scale(scale) * kLog2e;
    const int half = wave >> 1;   // of every stage: its keys 32 half ..
    PanelOffsets<D> fo;
    fo.init(fresh_lane(), half);
    const int wave_row0 = it.row0 + 64 * (wave & 1);
    const bool wave_active = has_rows(it, wave);   // (a scalar branch)
    const int wave_last_row = min(it.row0 + 64 * (wave & 1) + 63, it.doc_end - 1);
    const int n_steps = it.step_end - it.step_begin;
    const unsigned lds = lds_addr_of(smem) + wave * 1024;
    const int kv_first = it.doc_start + kStep * it.step_begin;
    {
      const bf16x8 zeros = zero_frag();
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < DB; ++i) acc_zero(acc[b][i], zeros);
    }
    // (as instructions that the compiler sees: for the statistics' loads it would wait, with all that is in flight by then,
    // inside the loop)
    if (follows) __builtin_amdgcn_s_waitcnt(0x0F70 + D / 16);
    else wait_all_vm_visible();
    __syncthreads();
    if (__builtin_expect(score_fold(scale) != 1.0f, 0)) FixedTiles<D>::fold(smem, wave, score_fold(scale));
    bf16x8 qf[2][KK], dof[2][KK];
    if (wave_active) FixedTiles<D>::read(smem, fo, wave, qf, dof);
    f32x16 s_init[2], dp_init[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      pin_frags_acc(qf[b]);
      pin_frags_acc(dof[b]);
      s_init[b] = f32x16(neg_lse_row[b]);
      dp_init[b] = f32x16(neg_dsum_row[b]);
      asm volatile("" : "+v"(s_init[b]), "+v"(dp_init[b]));
    }
    bf16x8 ka[KK];   // row fragments of K, read ahead
    int st = 0;
    auto stage = [&](int kv0, auto masked_c) __attribute__((always_inline)) {
      constexpr bool MASKED = decltype(masked_c)::value;
      const char* const kt = smem;
      const char* const vt = smem + kStage / 2;
      const unsigned next_lds = lds + (st & 1) * kStage, next_off = stream.offset();
      bf16x8 va[KK], tk[2][DB], dsb[2][2];
      f32x16 s[2], dp[2];
      int t_hi = 0;   // of block 0, allowed: 8 (r / 4) + r % 4 <= t_hi
      if constexpr (MASKED) {
        const int lane = fresh_lane();
        t_hi = wave_row0 - kv0 + (lane & 31) - 4 * (lane >> 5);
      }
      // 32 probabilities, block 0 then 1; 32 products with dP
      auto p_items = [&](auto first_c, auto last_c) __attribute__((always_inline)) {
#pragma unroll
        for (int i = decltype(first_c)::value; i < decltype(last_c)::value; ++i) {
          const int b = i >> 4, r = i & 15;
          float e = __builtin_amdgcn_exp2f(s[b][r] * cs);
          if (MASKED) {
            if (8 * (r >> 2) + (r & 3) > (b ? t_hi + (half ? -32 : 32) : t_hi)) e = 0.f;
          }
          s[b][r] = e;
        }
      };
      auto ds_items = [&](auto first_c, auto last_c) __attribute__((always_inline)) {
#pragma unroll
        for (int i = decltype(first_c)::value; i < decltype(last_c)::value; ++i) {
          const int b = i >> 4, r = i & 15;
          s[b][r] *= dp[b][r];
          if (r & 1) {
            const f32x2 ds = {s[b][r - 1], s[b][r]};
            const bf16x2 ds2 = __builtin_convertvector(ds, bf16x2);
            dsb[b][r >> 3][(r & 7) - 1] = ds2[0];
            dsb[b][r >> 3][r & 7] = ds2[1];
          }
        }
      };
      auto fence = []() __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };
      // vector work beside matrix instruction u of the 32 of S(1), dP(0), dP(1) and dQ(0) (the results of a phase are there two
      // instructions on)
      auto beside = [&](auto u_c) __attribute__((always_inline)) {
        constexpr int u = decltype(u_c)::value;
        auto share = [](int n, int from, int to, int at) { return at <= from ? 0 : at >= to ? n : n * (at - from) / (to - from); };
        constexpr int p_mid = KK + (KK == 8 ? 3 : 2), p_end = 3 * KK - (KK == 8 ? 2 : 1);
        constexpr int p0 = share(16, 2, p_mid, u) + share(16, p_mid, p_end, u), p1 = share(16, 2, p_mid, u + 1) + share(16, p_mid, p_end, u + 1);
        constexpr int d0 = share(16, 2 * KK + 2, 3 * KK, u) + share(16, 3 * KK + 2, 4 * KK, u);
        constexpr int d1 = share(16, 2 * KK + 2, 3 * KK, u + 1) + share(16, 3 * KK + 2, 4 * KK, u + 1);
        p_items(std::integral_constant<int, p0>{}, std::integral_constant<int, p1>{});
        ds_items(std::integral_constant<int, d0>{}, std::integral_constant<int, d1>{});
      };
      static_for<KK>([&](auto kk_c) {
        constexpr int kk = decltype(kk_c)::value;
        stream.template aim_piece<kk>(next_lds);
        if constexpr (kk == 0) mfma_vgpr_agpr_from(s[0], ka[kk], qf[0][kk], s_init[0]);
        else mfma_vgpr_agpr(s[0], ka[kk], qf[0][kk]);
        fence();
        stream.template load_piece<kk>(next_off);
        fence();
      });
      static_for<KK>([&](auto kk_c) {
        constexpr int kk = decltype(kk_c)::value;
        if constexpr (kk == 0) mfma_vgpr_agpr_from(s[1], ka[kk], qf[1][kk], s_init[1]);
        else mfma_vgpr_agpr(s[1], ka[kk], qf[1][kk]);
        va[kk] = fo.row_frag(vt, kk);
        beside(std::integral_constant<int, kk>{});
        fence();
      });
      static_for<KK>([&](auto kk_c) {
        constexpr int kk = decltype(kk_c)::value;
        if constexpr (kk == 0) mfma_vgpr_agpr_from(dp[0], va[kk], dof[0][kk], dp_init[0]);
        else mfma_vgpr_agpr(dp[0], va[kk], dof[0][kk]);
        beside(std::integral_constant<int, KK + kk>{});
        fence();
      });
      static_for<KK>([&](auto kk_c) {
        constexpr int kk = decltype(kk_c)::value;
        if constexpr (kk == 0) mfma_vgpr_agpr_from(dp[1], va[kk], dof[1][kk], dp_init[1]);
        else mfma_vgpr_agpr(dp[1], va[kk], dof[1][kk]);
        tk[kk / DB][kk % DB] = fo.trans_frag(kt, kk / DB, kk % DB);
        beside(std::integral_constant<int, 2 * KK + kk>{});
        fence();
      });
      static_for<2 * DB>([&](auto j_c) {
        constexpr int j = decltype(j_c)::value;
        acc[0][j % DB] = mfma(tk[j / DB][j % DB], dsb[0][j / DB], acc[0][j % DB]);
        beside(std::integral_constant<int, 3 * KK + j>{});
        fence();
      });
      wait_vm<0>();
      __syncthreads();
      fo.flip();
      // For the upper half of a diagonal stage block 1 lies in front of the keys: left out, not multiplied by zeros, so that an infinity
      // or NaN in K or V reaches dQ of the 31 rows in front of its token at most, as in bwd_dq_kernel.
      static_for<2 * DB>([&](auto j_c) {
        constexpr int j = decltype(j_c)::value;
        if (!MASKED || !half) acc[1][j % DB] = mfma(tk[j / DB][j % DB], dsb[1][j / DB], acc[1][j % DB]);
        ka[j] = fo.row_frag(smem, j);
        fence();
      });
    };
    // steps that hold a key for this wave: all but the last one of the diagonal (none where the chunk begins behind its rows)
    const int my_steps = wave_active ? min(n_steps, (wave_last_row - kv_first + kStep) / kStep) : 0;
    auto to_next = [&]() __attribute__((always_inline)) {   // the last step requests its own stage again (nobody reads it)
      const int kv0 = kv_first + kStep * st;
      if (++st < n_steps) {
        stream.advance();
        stream.aim(kv0 + kStep, it.doc_end - 1);
      }
      if (st >= n_steps - 1) tickets.step(st - (n_steps - 1));   // (not reached with 0 where there is one step)
      return kv0;
    };
    if (my_steps > 0) {
      static_for<KK>([&](auto kk) __attribute__((always_inline)) { ka[kk] = fo.row_frag(smem, kk); });
#pragma unroll 1
      do {
        const int kv0 = to_next();
        if (by_exec_mask(kv0 + kStep - 1 > wave_row0)) stage(kv0, std::true_type{});
        else stage(kv0, std::false_type{});
      } while (st < my_steps);
    }
#pragma unroll 1
    while (st < n_steps) {
      to_next();
      stream.load_stage(lds + (st & 1) * kStage);
      wait_vm<0>();
      __syncthreads();
    }
  }
};

// behind give(acc[1])
template <int D>
__device__ __forceinline__ void store_dq(const BwdArgs<D>& a, const varlen_attn_unit& it, int head, char* smem, int wave, const f32x16 (&acc)[2][D / 32]) {
  if (__builtin_expect(lower_half_only(it, false), 0)) {   // (one step: not cut)
    if (wave == 0) {
      uint2 w[D / 8];
      float mine[D / 32][16];
      static_for<D / 32>([&](auto db) __attribute__((always_inline)) { acc_values<db>(acc[0][db], mine[db]); });
      pack<D>(w, mine, a.scale);
      store_bf16<D>(smem, wave, fresh_lane(), it, w, a.dq, a.Hq, head);
    }
    return;
  }
  if (!has_rows(it, wave)) {
    skip_take();
    return;
  }
  const int lane = fresh_lane();
  f32x4 x[D / 8];
  float mine[D / 32][16];
  take<D, 0>(smem, wave, lane, acc[0], x, mine);
  add<D>(x, mine);
  if (it.slot >= 0) {
    store_partial<D>(a.row_partials + ((size_t)it.slot * a.Hq + head) * frag_floats<D>(), wave, lane, x);
  } else {
    uint2 w[D / 8];
#pragma unroll
    for (int i = 0; i < D / 8; ++i) w[i] = pack4(x[i][0] * a.scale, x[i][1] * a.scale, x[i][2] * a.scale, x[i][3] * a.scale);
    store_bf16<D>(smem, wave, lane, it, w, a.dq, a.Hq, head);
  }
}

template <int D>
struct DkvUnit {
  static constexpr int KK = D / 16, DB = D / 32, kStage = BwdLds<D>::kStage, kStat = BwdLds<D>::kStat;
  varlen_attn_unit it;
  int head, kvh;       // the first of the `hpu` q heads of a group that the unit sweeps one after the other; their kv head
  PanelStream<D> stream;
  unsigned long long stat_next;
  int stat_last, lane;
  float first_stat;    // of the unit's first stage, this lane's and wave's (in LDS they would lie where the results before meet)

  __device__ __forceinline__ void aim(int q0) {
    stream.aim(q0, it.doc_end - 1);
    stat_last = min(it.doc_end - 1 - q0, kStep - 1);
  }
  __device__ __forceinline__ void start(const BwdArgs<D>& a, int h, int wave) {   // at the first step of the chain, q head h
    const int q0 = it.row0 + kStep * it.step_begin;
    const size_t first = ((size_t)q0 * a.Hq + h) * D;
    stream.start(a.q + first, a.d_o + first);
    stat_next = uniform64((wave & 1 ? a.neg_dsum : a.neg_lse) + (size_t)h * a.N + q0);
    aim(q0);
  }
  __device__ __forceinline__ void load_stats(unsigned stat_lds) const { dma4(stat_next, (unsigned)min(lane, stat_last) * 4, stat_lds); }
  __device__ __forceinline__ void load_stage(char* smem, int wave, int b) const {   // to buffer `b`
    stream.load_stage(lds_addr_of(smem) + wave * 1024 + b * kStage);
    load_stats(stat_lds(smem, wave, b));
  }
  static __device__ __forceinline__ unsigned stat_lds(char* smem, int wave, int b) {
    return lds_addr_of(smem) + BwdLds<D>::kStats + (wave >> 1) * kStat + (wave & 1) * 256 + b * 2 * kStat;
  }
  __device__ __forceinline__ void open(const BwdArgs<D>& a, const varlen_attn_unit& unit, int head_, int kvh_, int hpu, char* smem, int wave, Tickets& tickets) {
    it = unit;
    head = head_;
    if (it.step_end - it.step_begin == 1 && hpu == 1) tickets.step(0);
    kvh = kvh_;
    lane = fresh_lane();
    stream.init(wave, lane, (unsigned)((size_t)a.Hq * D * 2));
    start(a, head, wave);
    stream.load_stage(lds_addr_of(smem) + wave * 1024);
    first_stat = reinterpret_cast<const float*>(stat_next)[min(lane, stat_last)];
    const size_t first = ((size_t)it.row0 * a.Hkv + kvh) * D;
    FixedTiles<D>::request(a.k + first, a.v + first, (unsigned)(a.Hkv * D * 2), it.row0, it.doc_end - 1, smem, wave);
  }

  // S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS.  `follows`: as in DqUnit, D / 8 stores.
  template <typename Tickets>
  __device__ __forceinline__ void sweep(const BwdArgs<D>& a, bool follows, int hpu, char* smem, int wave, f32x16 (&dkacc)[2][DB],
                                        f32x16 (&dvacc)[2][DB], Tickets& tickets) {
    float scale = a.scale;
    asm volatile("" : "+s"(scale));
    const float cs = folded_scale(scale) * kLog2e;
    const int half = wave >> 1;   // of every stage: its queries 32 half ..
    PanelOffsets<D> fo;
    fo.init(lane, half);
    const int wave_kv0 = it.row0 + 64 * (wave & 1);
    const bool wave_active = has_rows(it, wave);   // (a scalar branch)
    const int n_steps = it.step_end - it.step_begin;
    const unsigned lds = lds_addr_of(smem) + wave * 1024;
    {
      const bf16x8 zeros = zero_frag();
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < DB; ++i) { acc_zero(dkacc[b][i], zeros); acc_zero(dvacc[b][i], zeros); }
    }
    if (follows) __builtin_amdgcn_s_waitcnt(D == 128 ? 0x4F70 : 0x0F78);   // vmcnt(D / 8)
    else wait_all_vm_visible();
    *reinterpret_cast<float*>(smem + (stat_lds(smem, wave, 0) - lds_addr_of(smem)) + 4 * lane) = first_stat;
    __syncthreads();
    if (__builtin_expect(score_fold(scale) != 1.0f, 0)) FixedTiles<D>::fold(smem, wave, score_fold(scale));
    bf16x8 kf[2][KK], vf[2][KK];
    if (wave_active) FixedTiles<D>::read(smem, fo, wave, kf, vf);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      pin_frags(kf[b]);
      pin_frags(vf[b]);
    }

    // read ahead of a stage, behind the last matrix phase of the stage before it
    constexpr int kAhead = KK / 2;
    int stat_off = BwdLds<D>::kStats + half * (kStat + 128) + 16 * (lane >> 5);
    auto flip = [&]() __attribute__((always_inline)) { fo.flip(); stat_off ^= 2 * kStat; };   // to the other stage
    bf16x8 qa[kAhead];
    f32x16 s1;   // from -LSE / scale
    auto read_ahead = [&](auto i_c) __attribute__((always_inline)) {   // one of DB turns
      constexpr int i = decltype(i_c)::value;
#pragma unroll
      for (int rq = 4 / DB * i; rq < 4 / DB * (i + 1); ++rq) set4(s1, rq, *reinterpret_cast<const f32x4*>(smem + stat_off + 32 * rq));
      qa[i] = fo.row_frag(smem, i);
    };
    static_assert(kAhead == DB, "a fragment a turn");
    int heads_left = hpu, st = 0;
    auto stage = [&](int q0, auto masked_c) __attribute__((always_inline)) {
      constexpr bool MASKED = decltype(masked_c)::value;
      const char* const qt = smem;
      const char* const dot = smem + kStage / 2;
      const unsigned next_lds = lds + (st & 1) * kStage, next_off = stream.offset();
      bf16x8 q[KK], d[KK], tq[2][DB], td[2][DB], pb[2][2], dsb[2][2];
      f32x16 s0, dp0, dp1;
      int t_lo = 0, t_hi = 0;   // block 0, allowed: t_lo <= 8 (r / 4) + r % 4 < t_hi
      if constexpr (MASKED) {
        const int lane = fresh_lane(), h4 = 4 * (lane >> 5);
        t_lo = wave_kv0 - q0 + (lane & 31) - h4;
        t_hi = it.doc_end - q0 - 32 * half - h4;
      }
      auto fence = []() __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };
      auto p_item = [&](f32x16& sv, bf16x8 (&out)[2], int b, int r) __attribute__((always_inline)) {
        float e = __builtin_amdgcn_exp2f(sv[r] * cs);
        if (MASKED) {
          const int t = 8 * (r >> 2) + (r & 3);
          if (t < (b ? t_lo + (half ? -32 : 32) : t_lo) || t >= t_hi) e = 0.f;
        }
        sv[r] = e;
        if (r & 1) {
          const f32x2 p = {sv[r - 1], e};
          const bf16x2 p2 = __builtin_convertvector(p, bf16x2);
          out[r >> 3][(r & 7) - 1] = p2[0];
          out[r >> 3][r & 7] = p2[1];
        }
      };
      auto ds_item = [&](f32x16& sv, const f32x16& dpv, bf16x8 (&out)[2], int r) __attribute__((always_inline)) {
        sv[r] *= dpv[r];
        if (r & 1) {
          const f32x2 ds = {sv[r - 1], sv[r]};
          const bf16x2 ds2 = __builtin_convertvector(ds, bf16x2);
          out[r >> 3][(r & 7) - 1] = ds2[0];
          out[r >> 3][r & 7] = ds2[1];
        }
      };
      // vector work beside matrix instruction u of the 48 of dP, dV and dK: probabilities, then products, in the order in which the sums
      // take them: registers 0 .. 7 of block 0, of block 1, then 8 .. 15 (the results of a phase are there two instructions on)
      auto beside = [&](auto u_c) __attribute__((always_inline)) {
        constexpr int u = decltype(u_c)::value;
        auto share = [](int n, int from, int to, int at) { return at <= from ? 0 : at >= to ? n : n * (at - from) / (to - from); };
        constexpr int p_first = share(32, 2, 3 * KK - 1, u), p_last = share(32, 2, 3 * KK - 1, u + 1);
        constexpr int d_first = share(32, 3 * KK - 2, 5 * KK - 2, u), d_last = share(32, 3 * KK - 2, 5 * KK - 2, u + 1);
#pragma unroll
        for (int i = p_first; i < p_last; ++i) {
          const int r = (i & 7) + 8 * (i >> 4);
          if (i & 8) p_item(s1, pb[1], 1, r); else p_item(s0, pb[0], 0, r);
        }
#pragma unroll
        for (int i = d_first; i < d_last; ++i) {
          const int r = (i & 7) + 8 * (i >> 4);
          if (i & 8) ds_item(s1, dp1, dsb[1], r); else ds_item(s0, dp0, dsb[0], r);
        }
      };
      // transposed fragments in the order of their use, dO then Q, asked for kAheadT pairs of matrix instructions in front of it
      constexpr int kAheadT = 3;
      auto next_trans = [&](auto at_c) __attribute__((always_inline)) {
        constexpr int i = decltype(at_c)::value + kAheadT;
        if constexpr (i < 2 * DB) td[i / DB][i % DB] = fo.trans_frag(dot, i / DB, i % DB);
        else tq[i / DB - 2][i % DB] = fo.trans_frag(qt, i / DB - 2, i % DB);
      };
#pragma unroll
      for (int i = 0; i < kAhead; ++i) q[i] = qa[i];
      static_for<KK>([&](auto kk_c) {
        constexpr int kk = decltype(kk_c)::value;
        stream.template aim_piece<kk>(next_lds);
        if constexpr (kk == 0) mfma_vgpr_from(s0, q[kk], kf[0][kk], s1);
        else mfma_vgpr(s0, q[kk], kf[0][kk]);
        if constexpr (kk < kAhead) q[kk + kAhead] = fo.row_frag(qt, kk + kAhead);
        else d[kk - kAhead] = fo.row_frag(dot, kk - kAhead);
        fence();
        stream.template load_piece<kk>(next_off);
        if constexpr (kk == KK - 1) load_stats(stat_lds(smem, wave, st & 1));
        fence();
        mfma_vgpr(s1, q[kk], kf[1][kk]);
        if constexpr (kk < 4) set4(dp1, kk, *reinterpret_cast<const f32x4*>(smem + stat_off + 256 + 32 * kk));
        fence();
      });
      static_for<KK>([&](auto kk_c) {
        constexpr int kk = decltype(kk_c)::value;
        if constexpr (kk == 0) mfma_vgpr_from(dp0, d[kk], vf[0][kk], dp1);
        else mfma_vgpr(dp0, d[kk], vf[0][kk]);
        if constexpr (kk < kAhead) d[kk + kAhead] = fo.row_frag(dot, kk + kAhead);
        if constexpr (kk >= KK - kAheadT) next_trans(std::integral_constant<int, kk - KK>{});
        beside(std::integral_constant<int, 2 * kk>{});
        fence();
        mfma_vgpr(dp1, d[kk], vf[1][kk]);
        beside(std::integral_constant<int, 2 * kk + 1>{});
        fence();
      });
      static_for<2 * DB>([&](auto j_c) {
        constexpr int j = decltype(j_c)::value, cc = j / DB, db = j % DB;
        dvacc[0][db] = mfma(td[cc][db], pb[0][cc], dvacc[0][db]);
        next_trans(j_c);
        beside(std::integral_constant<int, 2 * KK + 2 * j>{});
        fence();
        dvacc[1][db] = mfma(td[cc][db], pb[1][cc], dvacc[1][db]);
        beside(std::integral_constant<int, 2 * KK + 2 * j + 1>{});
        fence();
      });
      static_for<2 * DB>([&](auto j_c) {
        constexpr int j = decltype(j_c)::value, cc = j / DB, db = j % DB;
        if constexpr (j == DB) {
          wait_vm<0>();
          __syncthreads();
          flip();
        }
        dkacc[0][db] = mfma(tq[cc][db], dsb[0][cc], dkacc[0][db]);
        if constexpr (j < DB) {
          if constexpr (2 * j < 2 * DB - kAheadT) next_trans(std::integral_constant<int, 2 * DB + 2 * j>{});
          beside(std::integral_constant<int, 4 * KK + 2 * j>{});
        } else {
          read_ahead(std::integral_constant<int, db>{});
        }
        fence();
        dkacc[1][db] = mfma(tq[cc][db], dsb[1][cc], dkacc[1][db]);
        if constexpr (j < DB) {
          if constexpr (2 * j + 1 < 2 * DB - kAheadT) next_trans(std::integral_constant<int, 2 * DB + 2 * j + 1>{});
          beside(std::integral_constant<int, 4 * KK + 2 * j + 1>{});
        }
        fence();
      });
    };
    auto to_next = [&]() __attribute__((always_inline)) {   // the last step requests its own stage again (nobody reads it)
      const int q0 = it.row0 + kStep * (it.step_begin + st);
      if (++st < n_steps) {
        stream.advance();
        stat_next += kStep * 4;
        aim(q0 + kStep);
      }
      if (st >= n_steps - 1 && heads_left == 1) tickets.step(st - (n_steps - 1));
      return q0;
    };
    auto idle = [&]() __attribute__((always_inline)) {   // a step without keys that its queries may see: loads and barrier only
      to_next();
      load_stage(smem, wave, st & 1);
      wait_vm<0>();
      __syncthreads();
      flip();
    };
    // every query of a chain's first step lies before the upper 64 keys
    const int begin = it.step_begin == 0 && (wave & 1) ? 1 : 0;
#pragma unroll 1
    for (;;) {
      if (begin) idle();
      if (wave_active && st < n_steps) {
        static_for<kAhead>([&](auto i) __attribute__((always_inline)) { read_ahead(i); });
#pragma unroll 1
        do {
          const int q0 = to_next();
          if (by_exec_mask(q0 < wave_kv0 + 64 || q0 + kStep > it.doc_end)) stage(q0, std::true_type{});
          else stage(q0, std::false_type{});
        } while (st < n_steps);
      }
#pragma unroll 1
      while (st < n_steps) idle();
      if (--heads_left == 0) break;
      __syncthreads();   // the last stage's read-ahead
      start(a, head + hpu - heads_left, wave);
      if (st & 1) flip();
      st = 0;
      if (n_steps == 1 && heads_left == 1) tickets.step(0);
      load_stage(smem, wave, 0);
      wait_vm<0>();
      __syncthreads();
    }
  }
};

// behind give(dkacc[1])
template <int D>
__device__ __forceinline__ void store_dkv(const BwdArgs<D>& a, const varlen_attn_unit& it, int head, int kvh, char* smem, int wave,
                                          const f32x16 (&dkacc)[2][D / 32], const f32x16 (&dvacc)[2][D / 32]) {
  constexpr int DB = D / 32;
  if (__builtin_expect(lower_half_only(it, true), 0)) {
    if (wave == 0) {
      const int lane = fresh_lane();
      uint2 w[D / 8];
      float mine[DB][16];
      static_for<DB>([&](auto db) __attribute__((always_inline)) { acc_values<db>(dkacc[0][db], mine[db]); });
      if (it.slot >= 0) {
        float* const partial = a.col_partials + ((size_t)it.slot * a.Hq + head) * 2 * frag_floats<D>();
        store_partial<D>(partial, mine, lane);
        static_for<DB>([&](auto db) __attribute__((always_inline)) { acc_values<2 * DB + db>(dvacc[0][db], mine[db]); });
        store_partial<D>(partial + frag_floats<D>(), mine, lane);
      } else {
        pack<D>(w, mine, a.scale);
        store_bf16<D>(smem, wave, lane, it, w, a.dk, a.Hkv, kvh);
        static_for<DB>([&](auto db) __attribute__((always_inline)) { acc_values<2 * DB + db>(dvacc[0][db], mine[db]); });
        pack<D>(w, mine, 1.f);
        store_bf16<D>(smem, wave, lane, it, w, a.dv, a.Hkv, kvh);
      }
    }
    return;
  }
  if (!has_rows(it, wave)) {
    skip_take();
    skip_take();
    return;
  }
  const int lane = fresh_lane();
  float* const partial = a.col_partials + ((size_t)it.slot * a.Hq + head) * 2 * frag_floats<D>();
  f32x4 x[D / 8];
  float mine[DB][16];
  uint2 dk[D / 8], dv[D / 8];
  take<D, 0>(smem, wave, lane, dkacc[0], x, mine);
  give<D, 3 * DB>(smem, wave, true, dvacc[1]);   // on its way to LDS while dK is dealt with
  add<D>(x, mine);
  if (it.slot >= 0) {
    store_partial<D>(partial, wave, lane, x);
  } else {
#pragma unroll
    for (int i = 0; i < D / 8; ++i) dk[i] = pack4(x[i][0] * a.scale, x[i][1] * a.scale, x[i][2] * a.scale, x[i][3] * a.scale);
  }
  take<D, 2 * DB>(smem, wave, lane, dvacc[0], x, mine);
  add<D>(x, mine);
  if (it.slot >= 0) {
    store_partial<D>(partial + frag_floats<D>(), wave, lane, x);
  } else {
    store_bf16<D>(smem, wave, lane, it, dk, a.dk, a.Hkv, kvh);
#pragma unroll
    for (int i = 0; i < D / 8; ++i) dv[i] = pack4(x[i][0], x[i][1], x[i][2], x[i][3]);
    store_bf16<D>(smem, wave, lane, it, dv, a.dv, a.Hkv, kvh);
  }
}

template <int D>
__global__ void __launch_bounds__(kThreads, 1) bwd_pool_kernel(BwdArgs<D>) {
  // The arguments are fetched anew for every unit (scalar loads): kept across the units they would be spilled.
  auto fresh = []() __attribute__((always_inline)) {
    auto p = (const __attribute__((address_space(4))) BwdArgs<D>*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const BwdArgs<D>*)p;
  };
  const BwdArgs<D> a = fresh();
  __shared__ __attribute__((aligned(1024))) char smem[BwdLds<D>::kBytes];
  // the units do not change while the kernel runs: scalar loads
  typedef const __attribute__((address_space(4))) varlen_attn_unit* constant_units;
  auto load_unit = [&](const varlen_attn_unit* units, int i) __attribute__((always_inline)) {
    const constant_units u = (constant_units)(size_t)units;
    return varlen_attn_unit{u[i].row0, u[i].doc_start, u[i].doc_end, u[i].step_begin, u[i].step_end, u[i].slot, 0, 0};
  };
  // the first unit where column units take one q head, fetched together with the header that says so
  TicketGroup g;
  g.init(blockIdx.x, gridDim.x, a.Hq, 1);
  const varlen_attn_unit early = load_unit(a.col_units, min(g.heads(g.first), a.max_units - 1));
  const int hpu = a.hdr->col_heads_per_unit, n_col = a.hdr->n_col_units;
  // a plan that was made for two kernels has no dQ units of its own: the row units
  const bool own_dq = a.hdr->n_dq_units > 0;
  const int n_dq = own_dq ? a.hdr->n_dq_units : a.hdr->n_row_units;
  if (n_col == 0) return;   // nothing planned
  if (hpu != 1) g.init(blockIdx.x, gridDim.x, a.Hq, hpu);
  g.set(n_col, n_dq);
  if (g.first >= g.total) return;
  Divisor group;   // q heads of a kv head
  group.init(a.Hq / a.Hkv);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Tickets tickets{a.tickets + g.index, reinterpret_cast<int*>(smem + BwdLds<D>::kTicket), 0};
  DqUnit<D> row;
  int t = g.first, unit, head;
  g.decode(t, unit, head);
  if (t < g.n_col) {
    DkvUnit<D> col;
    col.open(a, hpu == 1 ? early : load_unit(a.col_units, unit), head, group(head), hpu, smem, wave, tickets);
    f32x16 dkacc[2][D / 32], dvacc[2][D / 32];
#pragma unroll 1
    for (bool follows = false;;) {
      col.sweep(a, follows, hpu, smem, wave, dkacc, dvacc, tickets);
      const varlen_attn_unit done = col.it;
      const int done_head = col.head, done_kvh = col.kvh;
      t = g.members + tickets.take();
      const bool meet = !lower_half_only(done, true);
      follows = has_rows(done, wave) && (meet || wave == 0);
      give<D, D / 32>(smem, wave, follows && meet, dkacc[1]);
      g.decode(t, unit, head);
      const BwdArgs<D> b = fresh();
      if (t < g.n_col) col.open(b, load_unit(b.col_units, unit), head, group(head), hpu, smem, wave, tickets);
      store_dkv<D>(b, done, done_head, done_kvh, smem, wave, dkacc, dvacc);
      if (t >= g.n_col) break;
    }
    if (t >= g.total) return;
  }
  {
    const BwdArgs<D> b = fresh();
    row.open(b, load_unit(own_dq ? b.dq_units : b.row_units, unit), head, group(head), smem, wave, tickets);
  }
  f32x16 acc[2][D / 32];
#pragma unroll 1
  for (bool follows = false;;) {
    row.sweep(a, follows, smem, wave, acc, tickets);
    const varlen_attn_unit done = row.it;
    const int done_head = row.head;
    t = g.members + tickets.take();
    const bool meet = !lower_half_only(done, false);
    follows = has_rows(done, wave) && (meet || wave == 0);
    give<D, D / 32>(smem, wave, follows && meet, acc[1]);
    const BwdArgs<D> b = fresh();
    if (t < g.total) {
      g.decode(t, unit, head);
      row.open(b, load_unit(own_dq ? b.dq_units : b.row_units, unit), head, group(head), smem, wave, tickets);
    }
    store_dq<D>(b, done, done_head, smem, wave, acc);
    if (t >= g.total) break;
  }
}

// Sums of the partial results of the pool, dealt as in fwd_combine_kernel: [dK | dV] of cut or grouped column tiles by the
// workgroups from the front, dQ of cut tiles of the units it came from (dQ units or, where the plan has none, row units) by
// the workgroups from the back.
template <int D>
__global__ void __launch_bounds__(kThreads)
bwd_pool_combine_kernel(const varlen_attn_plan_header* __restrict__ hdr, const varlen_attn_combine_item* __restrict__ col_items,
                        int max_col, const float* __restrict__ col_partials, const varlen_attn_combine_item* __restrict__ dq_items,
                        const varlen_attn_combine_item* __restrict__ row_items, int max_row, const float* __restrict__ row_partials, __bf16* __restrict__ dq, __bf16* __restrict__ dk,
                        __bf16* __restrict__ dv, int Hq, int Hkv, float scale) {
  constexpr int DB = D / 32, kWavePieces = 4 * DB / 2;
  constexpr int kFlight = 4;
  using Tile = RowTile<64>;
  __shared__ __attribute__((aligned(16))) char tiles[2][Tile::kBytes];
  int buf = 0;
  const int lane = threadIdx.x & 63, rq = threadIdx.x >> 6, h = lane >> 5, c = lane & 31;
  const int n_col = min(hdr->n_col_combine, max_col), hpu = hdr->col_heads_per_unit;
  const bool own_dq = hdr->n_dq_units > 0;
  const int n_row = min(own_dq ? hdr->n_dq_combine : hdr->n_row_combine, max_row);
  if (!own_dq) dq_items = row_items;
  const int G = Hq / Hkv;
  auto piece = [&](const varlen_attn_combine_item& it, int wave, int db, const float* p0, int n_parts, auto offset, float mul, __bf16* out, int out_heads, int out_head)
      __attribute__((always_inline)) {
    const int row0 = it.row0 + 32 * wave;
    if (row0 >= it.doc_end) return;
    p0 += (size_t)(wave * DB + db) * kThreads * 4 + (size_t)threadIdx.x * 4;
    f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
#pragma unroll 1
    for (int j0 = 0; j0 < n_parts; j0 += kFlight) {
      f32x4 xa[kFlight], xb[kFlight];
#pragma unroll
      for (int j = 0; j < kFlight; ++j) {
        xa[j] = xb[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (j0 + j < n_parts) {
          const size_t off = offset(j0 + j);
          xa[j] = *reinterpret_cast<const f32x4*>(p0 + off);
          xb[j] = *reinterpret_cast<const f32x4*>(p0 + off + kThreads * 4);
        }
      }
#pragma unroll
      for (int j = 0; j < kFlight; ++j) { acc0 += xa[j]; acc1 += xb[j]; }
    }
    Tile::put(tiles[buf], c, h, rq, pack4(acc0[0] * mul, acc0[1] * mul, acc0[2] * mul, acc0[3] * mul));
    Tile::put(tiles[buf], c, h, 4 + rq, pack4(acc1[0] * mul, acc1[1] * mul, acc1[2] * mul, acc1[3] * mul));
    __syncthreads();
    const int out_row = row0 + (threadIdx.x >> 3), chunk = threadIdx.x & 7;
    const uint4 w = Tile::get(tiles[buf], threadIdx.x >> 3, chunk);
    if (out_row < it.doc_end) *reinterpret_cast<uint4*>(out + ((size_t)out_row * out_heads + out_head) * D + 32 * db + 8 * chunk) = w;
    buf ^= 1;
  };
  constexpr size_t csize = 2 * frag_floats<D>(), rsize = frag_floats<D>();
#pragma unroll 1
  for (int work = blockIdx.x; work < n_col * Hkv * 2 * kWavePieces; work += gridDim.x) {
    const int tensor = work & 1, pc = (work >> 1) % kWavePieces, rest = (work >> 1) / kWavePieces;
    const int idx = rest / Hkv, oh = rest % Hkv;
    const varlen_attn_combine_item it = col_items[idx];
    const int Gp = G / hpu;
    piece(it, pc / (DB / 2), 2 * (pc % (DB / 2)), col_partials + ((size_t)it.slot0 * Hq + oh * G) * csize + tensor * frag_floats<D>(), it.n_chunks * Gp,
          [&](int j) { return ((size_t)(j / Gp) * Hq + (j % Gp) * hpu) * csize; }, tensor == 0 ? scale : 1.0f, tensor == 0 ? dk : dv, Hkv, oh);
  }
#pragma unroll 1
  for (int work = gridDim.x - 1 - blockIdx.x; work < n_row * Hq * kWavePieces; work += gridDim.x) {
    const int pc = work % kWavePieces, rest = work / kWavePieces;
    const int idx = rest / Hq, head = rest % Hq;
    const varlen_attn_combine_item it = dq_items[idx];
    piece(it, pc / (DB / 2), 2 * (pc % (DB / 2)), row_partials + ((size_t)it.slot0 * Hq + head) * rsize, it.n_chunks,
          [&](int j) { return (size_t)j * Hq * rsize; }, scale, dq, Hq, head);
  }
}

}  // namespace

#endif  // VARLEN_ATTN_BWD_POOL_HPP_
