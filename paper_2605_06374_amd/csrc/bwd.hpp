// Backward kernels (dQ; dK and dV) and the reduction of their partial results.
#ifndef VARLEN_ATTN_BWD_HPP_
#define VARLEN_ATTN_BWD_HPP_

#include "tiles.hpp"
#include "staging.hpp"
#include "fragments.hpp"
#include "plan.hpp"

namespace {

// ----------------------------------------------------------------------------------------
// Backward, dQ (first backward kernel).  Same decomposition as the forward: one workgroup per
// (row unit, q head).  Its prologue also computes D = rowsum(dO * O) for its rows.
// S^T = K Q^T, dP^T = V dO^T, dS^T = P^T (dP^T - D), dQ^T += K^T dS^T.
// ----------------------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(kThreads, 2)
bwd_dq_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k,
              const __bf16* __restrict__ v, const __bf16* __restrict__ o,
              const __bf16* __restrict__ d_o, const float* __restrict__ lse,
              float* __restrict__ neg_dsum, float* __restrict__ neg_lse,
              const varlen_attn_plan_header* __restrict__ hdr,
              const varlen_attn_unit* __restrict__ units, __bf16* __restrict__ dq,
              float* __restrict__ partials, int N, int Hq, int Hkv, float scale,
              int max_units) {
  constexpr int KK = D / 16, DB = D / 32;
  constexpr int NS = 4;
  constexpr int kStageBytes = kSub * D * 2;
  constexpr int LPS = PairStream<D, kSub>::kPieces;  // direct-to-LDS loads per wave and stage (K and V)
  static_assert(2 * LPS <= KK, "a load behind every other pair of matrix instructions");
  __shared__ __attribute__((aligned(1024))) char smem[2 * NS * kStageBytes];  // K stages, V stages

  int unit_idx, head;
  decode_block(blockIdx.x, Hq, unit_idx, head);
  // both loads in flight together; the unit array always has max_units >= grid / Hq entries
  const int n_units = hdr->n_row_units;
  const varlen_attn_unit it = units[min(unit_idx, max_units - 1)];
  if (unit_idx >= n_units) return;
  const int kvh = head / (Hq / Hkv);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, c = lane & 31;
  const float cs = scale * kLog2e;

  // (from the thread index: as in the dK/dV kernel the branches must stay exec-masked)
  const int wave_row0 = it.row0 + 32 * (tid >> 6);
  const int my_row = wave_row0 + c;
  const bool row_valid = my_row < it.doc_end;
  const bool wave_active = wave_row0 < it.doc_end;
  const int wave_last_row = min(wave_row0 + 31, it.doc_end - 1);
  const int wg_last_row = min(it.row0 + kTile, it.doc_end) - 1;
  const int kv_begin = it.doc_start + it.step_begin * kStep;
  const int kv_end = min(it.doc_start + it.step_end * kStep, wg_last_row + 1);
  const int n_sub = (kv_end - kv_begin + kSub - 1) / kSub;

  const __bf16* kbase = k + (size_t)kvh * D;
  const __bf16* vbase = v + (size_t)kvh * D;
  const size_t kv_stride = (size_t)Hkv * D;
  const unsigned lds_k = lds_addr_of(smem) + wave * 1024, lds_v = lds_k + NS * kStageBytes;

  // stages are requested in order: the wave-uniform addresses of the next stage's first K and V
  // rows live in scalar registers and move on by one stage per sub-step
  PairStream<D, kSub> stream;
  stream.init(wave, lane, (unsigned)(kv_stride * 2));
  stream.start(kbase + (size_t)kv_begin * kv_stride, vbase + (size_t)kv_begin * kv_stride);
  stream.aim(kv_begin, it.doc_end - 1);
  // past the last stage the last one is requested again (into a buffer that nobody reads), so that
  // every sub-step is the same
  auto next_stage = [&](int sub) __attribute__((always_inline)) {
    if (sub < n_sub) {
      stream.advance();
      stream.aim(kv_begin + kSub * sub, it.doc_end - 1);
    }
  };
  auto piece = [&](auto piece_c, auto stage_c) __attribute__((always_inline)) {
    constexpr int P = decltype(piece_c)::value, ST = decltype(stage_c)::value;
    stream.template piece<P>(lds_k + ST * kStageBytes, lds_v + ST * kStageBytes);
  };
  auto all_pieces = [&](auto stage_c) __attribute__((always_inline)) {
    static_for<LPS>([&](auto p) __attribute__((always_inline)) { piece(p, stage_c); });
  };
  static_for<NS - 1>([&](auto st) __attribute__((always_inline)) {
    if (st > 0) next_stage(st);
    all_pieces(st);
  });

  // Q and dO fragments stay in registers; the O fragments are only needed for
  // D = rowsum(dO * O): each lane holds half of its row's columns, the other half-wave the rest.
  bf16x8 qf[KK], dof[KK];
  const int load_row = min(my_row, it.doc_end - 1);   // rows past the document end: duplicates, never stored
  const size_t row_off = ((size_t)load_row * Hq + head) * D;
  float lse_row = lse[(size_t)head * N + load_row];
  float d_part = 0.f;
  {
    bf16x8 of[KK];
    load_row_frags<D>(d_o + row_off, h, dof);
    load_row_frags<D>(o + row_off, h, of);
    load_row_frags<D>(q + row_off, h, qf);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int e = 0; e < 8; ++e) d_part += (float)dof[kk][e] * (float)of[kk][e];
  }
  const float dsum_row = half_sum(d_part);
  // rows past the document end get LSE = +huge so that their P is exactly 0
  if (!row_valid) lse_row = 1e30f;
  const float lse2 = lse_row * kLog2e;
  // the unit that starts the chain publishes -D and -LSE / scale for the dK/dV kernel
  if (it.step_begin == 0 && row_valid && h == 0) {
    neg_dsum[(size_t)head * N + my_row] = -dsum_row;
    neg_lse[(size_t)head * N + my_row] = -lse_row / folded_scale(scale);
  }
  FragOffsets<D> fo;
  fo.init(lane);
  wait_all_vm_visible();
  pin_frags(qf);
  pin_frags(dof);

  f32x16 acc[DB];
#pragma unroll
  for (int i = 0; i < DB; ++i) acc[i] = f32x16(0.f);

  auto compute = [&](int sub, auto stage_c) {
    constexpr int ST = decltype(stage_c)::value;
    const int kv0 = kv_begin + kSub * sub;
    const std::integral_constant<int, (ST + NS - 1) % NS> far_c{};
    if (!(wave_active && kv0 <= wave_last_row)) { all_pieces(far_c); return; }
    const char* kt = smem + ST * kStageBytes;
    const char* vt = smem + (NS + ST) * kStageBytes;
    f32x16 s = f32x16(0.f), dp = f32x16(0.f);
    __builtin_amdgcn_s_setprio(2);   // matrix phases win the issue slot over the other wave's vector work
    bf16x8 kf[KK], vf[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      kf[kk] = lds_read_frag(kt, fo.row_frag[kk]);
      vf[kk] = lds_read_frag(vt, fo.row_frag[kk]);
    }
    // one of the direct-to-LDS loads of the stage NS - 1 ahead behind every other pair, instead of
    // all of them behind the barrier: 555 -> 550 us at 32768 tokens in 11 documents, 38.9 -> 38.1 us
    // at 8192 tokens (the same in the forward, whose pairs of waves hide the clump, gives nothing)
    static_for<KK>([&](auto kk) __attribute__((always_inline)) {
      s = mfma(kf[kk], qf[kk], s);
      dp = mfma(vf[kk], dof[kk], dp);
      if constexpr (kk % 2 == 1 && kk / 2 < LPS) {
        __builtin_amdgcn_sched_barrier(0);
        piece(std::integral_constant<int, kk / 2>{}, far_c);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    __builtin_amdgcn_s_setprio(0);
    // the transposed K fragments of the last contraction are requested before the vector
    // work, so that they arrive behind it
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 ktf[2][DB];
#pragma unroll
    for (int cc = 0; cc < 2; ++cc)
#pragma unroll
      for (int db = 0; db < DB; ++db) ktf[cc][db] = read_trans<D>(kt, fo, cc, db);
    __builtin_amdgcn_sched_barrier(0);
    if (kv0 + kSub - 1 > wave_row0) {  // touches the diagonal for some row (wave-uniform)
      const int t = my_row - kv0 - 4 * h;  // key offset 8 (r / 4) + r % 4 is allowed iff <= t
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], cs, -lse2));
        if (8 * (r / 4) + (r % 4) > t) p = 0.f;
        s[r] = p * (dp[r] - dsum_row);
      }
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], cs, -lse2));
        s[r] = p * (dp[r] - dsum_row);
      }
    }
    __builtin_amdgcn_s_setprio(2);
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
      const bf16x8 dsb = pack8(s, 8 * cc);
#pragma unroll
      for (int db = 0; db < DB; ++db) acc[db] = mfma(ktf[cc][db], dsb, acc[db]);
    }
    __builtin_amdgcn_s_setprio(0);
  };
  auto body = [&](int sub, auto stage_c) {
    constexpr int ST = decltype(stage_c)::value;
    wait_vm<(NS - 2) * LPS>();
    __syncthreads();
    next_stage(sub + NS - 1);
    compute(sub, stage_c);
  };
  for (int sub = 0; sub < n_sub; sub += NS) {
    body(sub, std::integral_constant<int, 0>{});
    if (sub + 1 >= n_sub) break;
    body(sub + 1, std::integral_constant<int, 1>{});
    if (sub + 2 >= n_sub) break;
    body(sub + 2, std::integral_constant<int, 2>{});
    if (sub + 3 >= n_sub) break;
    body(sub + 3, std::integral_constant<int, 3>{});
  }
  wait_vm<0>();  // nothing may still be landing in LDS when the workgroup retires

  if (it.slot >= 0) {
    store_frag<D>(partials + ((size_t)it.slot * Hq + head) * frag_floats<D>(), acc, wave, lane);
    return;
  }
  __syncthreads();   // every wave is done with the stages
  store_rows<D>(smem + wave * RowTile<D>::kBytes, dq + ((size_t)wave_row0 * Hq + head) * D, (size_t)Hq * D,
                it.doc_end - wave_row0, acc, lane, scale);
}

// ----------------------------------------------------------------------------------------
// First kernel of the fused backward (VARLEN_ATTN_FLAG_FUSED_BWD) and of the pooled one (bwd_pool.hpp):
// -D = -rowsum(dO * O) and -LSE / scale for every (token, q head) into the workspace; the fp32 dQ accumulator
// (fused) or the ticket counters (pooled) cleared.  One group of D / 8 lanes per row (16 bytes per lane); bound by
// memory (67 MB in 13 us at 32768 tokens, 4 heads of 128; four rows a group took 1 us longer at 8192 tokens).
// ----------------------------------------------------------------------------------------
template <int D, bool FUSED>
__global__ void __launch_bounds__(kThreads)
bwd_prep_kernel(const __bf16* __restrict__ o, const __bf16* __restrict__ d_o,
                const float* __restrict__ lse, float* __restrict__ neg_dsum,
                float* __restrict__ neg_lse, float* __restrict__ dq_acc, int* __restrict__ tickets, int N, int Hq, float scale) {
  if (!FUSED && blockIdx.x == 0 && threadIdx.x < kTicketCounters) tickets[threadIdx.x] = 0;
  constexpr int kLanesPerRow = D / 8;
  constexpr int kRowsPerBlock = kThreads / kLanesPerRow;
  const long long row = (long long)blockIdx.x * kRowsPerBlock + threadIdx.x / kLanesPerRow;  // t * Hq + h
  const int part = threadIdx.x % kLanesPerRow;
  const bool valid = row < (long long)N * Hq;
  float acc = 0.f;
  if (valid) {
    const uint4 a = *reinterpret_cast<const uint4*>(d_o + row * D + 8 * part);
    const uint4 b = *reinterpret_cast<const uint4*>(o + row * D + 8 * part);
    const bf16x8 x = __builtin_bit_cast(bf16x8, a), y = __builtin_bit_cast(bf16x8, b);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc += (float)x[e] * (float)y[e];
    if (FUSED) {
      f32x4* z = reinterpret_cast<f32x4*>(dq_acc + row * D + 8 * part);
      z[0] = f32x4{0.f, 0.f, 0.f, 0.f};
      z[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
#pragma unroll
  for (int off = kLanesPerRow / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
  if (part == 0 && valid) {
    const int t = (int)(row / Hq), h = (int)(row % Hq);
    neg_dsum[(size_t)h * N + t] = -acc;
    neg_lse[(size_t)h * N + t] = -lse[(size_t)h * N + t] / folded_scale(scale);
  }
}

// Fused backward, last kernel: dQ = scale * accumulator, rounded to bf16.
template <int D>
__global__ void __launch_bounds__(kThreads)
bwd_dq_finish_kernel(const float* __restrict__ dq_acc, __bf16* __restrict__ dq, long long n8,
                     float scale) {
  const long long i = (long long)blockIdx.x * kThreads + threadIdx.x;   // group of 8 elements
  if (i >= n8) return;
  const f32x4 a = reinterpret_cast<const f32x4*>(dq_acc)[2 * i], b = reinterpret_cast<const f32x4*>(dq_acc)[2 * i + 1];
  const uint2 lo = pack4(a[0] * scale, a[1] * scale, a[2] * scale, a[3] * scale);
  const uint2 hi = pack4(b[0] * scale, b[1] * scale, b[2] * scale, b[3] * scale);
  reinterpret_cast<uint4*>(dq)[i] = uint4{lo.x, lo.y, hi.x, hi.y};
}

// Sum of the dQ partials of one cut tile and q head by one whole workgroup (thread t owns the
// float4s t, t + 256, ... of the fragment; chunks are added in chain order, as many loads in
// flight as four chunks of four float4s).  These workgroups ride at the end of the dK/dV
// kernel's grid: the dQ partials are complete when that kernel starts, and its last round
// leaves most compute units idle, so the reduction costs no launch and no time of its own.
template <int D>
__device__ __forceinline__ void dq_tile_combine(int block, const varlen_attn_plan_header* __restrict__ hdr,
                                                int max_items,
                                                const varlen_attn_combine_item* __restrict__ items,
                                                const float* __restrict__ partials,
                                                __bf16* __restrict__ dq, int Hq, float scale, char* lds) {
  constexpr int DB = D / 32;
  using Tile = RowTile<D>;
  constexpr int kTiles = 4 / DB;   // [32][D] tiles that four float4s of every thread make up
  constexpr int kPerThread = kTile * D / 4 / kThreads;   // float4s of a fragment per thread
  const int idx = block / Hq, head = block % Hq;
  // both loads in flight together
  const int n_items = hdr->n_row_combine;
  const varlen_attn_combine_item it = items[min(idx, max_items - 1)];
  if (idx >= n_items) return;
  const size_t pstride = (size_t)Hq * frag_floats<D>();
  const float* p0 = partials + ((size_t)it.slot0 * Hq + head) * frag_floats<D>() + (size_t)threadIdx.x * 4;
#pragma unroll 1
  for (int s0 = 0; s0 < kPerThread; s0 += 4) {
    f32x4 acc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int c0 = 0; c0 < it.n_chunks; c0 += 4) {
      f32x4 x[4][4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          x[j][u] = f32x4{0.f, 0.f, 0.f, 0.f};
          if (c0 + j < it.n_chunks)   // the same for the whole workgroup
            x[j][u] = *reinterpret_cast<const f32x4*>(p0 + (size_t)(c0 + j) * pstride +
                                                      (size_t)(s0 + u) * kThreads * 4);
        }
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (c0 + j < it.n_chunks) acc[u] += x[j][u];
    }
    // float4 s0 + u of a thread: wave (s0 + u) / DB, column block (s0 + u) % DB, register quad = the
    // thread's wave.  The rows are put together in LDS (two buffers in turn) and stored whole.
    char* const tiles = lds + ((s0 >> 2) & 1) * kTiles * Tile::kBytes;
    const int lane = threadIdx.x & 63, rq = threadIdx.x >> 6;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      Tile::put(tiles + (u / DB) * Tile::kBytes, lane & 31, lane >> 5, 4 * (u % DB) + rq,
                pack4(acc[u][0] * scale, acc[u][1] * scale, acc[u][2] * scale, acc[u][3] * scale));
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      constexpr int kRows = kThreads / Tile::kChunks;   // 16 or 32: per store of the workgroup
      const int row = kRows * i + threadIdx.x / Tile::kChunks, chunk = threadIdx.x % Tile::kChunks;
      const uint4 w = Tile::get(tiles + (row / 32) * Tile::kBytes, row % 32, chunk);
      const int out_row = it.row0 + 32 * (s0 / DB) + row;
      if (out_row < it.doc_end) *reinterpret_cast<uint4*>(dq + ((size_t)out_row * Hq + head) * D + 8 * chunk) = w;
    }
  }
}

// ----------------------------------------------------------------------------------------
// Backward, dK and dV.  One workgroup per (column unit, q head): wave w owns key rows
// row0 + 32w .. +31, keeps their K and V fragments in registers, and sweeps the unit's
// query steps (from the diagonal towards the document end).
//   S = Q K^T, dP = dO V^T (query rows in registers r, key on the lane),
//   dV^T += dO^T P,  dK^T += Q^T dS.
// What bounds it: at d = 128 one wave per SIMD issues everything, so that every instruction beside the
// matrix instructions costs; hence the direct-to-LDS loads of the next stage between the matrix
// instructions of M1(0) (a clump of 10 of them behind the barrier left the matrix pipe idle for some
// 250 clocks of a stage) and accumulators that start from -LSE / scale and -D (no subtractions):
// 824 -> 769 us at 32768 tokens in 11 documents (205e6 pairs, 4 heads of 128), 305 -> 283 us at 16384
// tokens with 8 q heads on one kv head.  The registers that the statistics no longer need let the
// d = 64 form run two workgroups per CU: 58.4 -> 40.6 us at 6144 tokens, 16 q and 4 kv heads.
// With grouped-query attention, or when the chain is cut, the unit stores fp32 partials
// [dK | dV] that bwd_combine_kernel adds up over the chunks and the q heads of the group.
//
// FUSED (VARLEN_ATTN_FLAG_FUSED_BWD): the kernel also forms dQ, so that S and dP are computed
// once for the whole backward (5 contractions instead of 7).  dS of a stage goes, as bf16, into
// an LDS tile [128 keys][64 queries]; one stage later wave w multiplies it with columns
// 32w .. 32w+31 of the unit's K tile (kept in LDS for this) and adds the 64 x 32 block of
// dQ = dS K into a fp32 accumulator in the workspace with floating-point atomics: the order of
// those additions is not fixed, so dQ is not bit-reproducible in this mode.  HALVES (heads of 128): dV is summed
// over the lower and over the upper 32 queries of the stages apart and then together, as the pool does (bwd_pool.hpp), so that it
// has the bits of the backward without the flag.
// ----------------------------------------------------------------------------------------
template <int D, bool FUSED, bool HALVES = false>
__global__ void __launch_bounds__(kThreads, D == 64 && !FUSED ? 2 : 1)
bwd_dkv_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k,
               const __bf16* __restrict__ v, const __bf16* __restrict__ d_o,
               const float* __restrict__ neg_lse, const float* __restrict__ neg_dsum,
               const varlen_attn_plan_header* __restrict__ hdr,
               const varlen_attn_unit* __restrict__ units, __bf16* __restrict__ dk,
               __bf16* __restrict__ dv, float* __restrict__ partials, int N, int Hq, int Hkv,
               float scale, int max_units, int unit_blocks,
               const varlen_attn_combine_item* __restrict__ row_items, int max_items,
               const float* __restrict__ row_partials, __bf16* __restrict__ dq,
               float* __restrict__ dq_acc) {
  constexpr int KK = D / 16, DB = D / 32;
  static_assert(KK == 2 * DB, "the phases of a stage have the same number of matrix instructions");
  // S and dP of the d = 128 form in vector registers: with more than 256 registers in use the
  // compiler puts every matrix result into accumulation registers, which the vector ALU cannot
  // read, and copies each score (64 of 426 instructions of a stage; 767 -> 733 us at 32768 tokens in
  // 11 documents, 285 -> 272 us at 16384 tokens, 8 q heads).
  constexpr bool kVgprScores = D == 128 && !FUSED;
  // The compiler does not see that these results take time: nothing may read them until two further
  // matrix instructions have been issued.  The softmax of a block therefore starts beside the third
  // matrix instruction of the phase behind it (SKEW), fences before and after.
  constexpr int SKEW = kVgprScores ? 2 : 0;
  auto mfma_s = [&](f32x16& c, const bf16x8& a, const bf16x8& b) __attribute__((always_inline)) {
    if constexpr (kVgprScores) mfma_vgpr(c, a, b);
    else c = mfma(a, b, c);
  };
  // Two stages of kStep = 64 query rows: one stage of lookahead is a whole stage of compute
  // (this kernel runs one workgroup per CU), and 64 KB of tiles keeps every LDS offset inside
  // the 16-bit immediate of the read instructions.
  constexpr int NS = 2;
  constexpr int kStageBytes = kStep * D * 2;
  constexpr int kStatBytes = 512;             // -LSE / scale [64] then -D [64]; two copies, one per pair of waves
  using Stream = PairStream<D, kStep>;
  static_assert(Stream::kPieces == KK, "one piece of the next stage beside each pair of matrix instructions");
  constexpr int kPlainBytes = 2 * NS * kStageBytes + NS * 2 * kStatBytes;
  constexpr int kKeyTileBytes = FUSED ? kTile * D * 2 : 0;      // the unit's K rows [128][D]
  constexpr int kDsBytes = FUSED ? kTile * kStep * 2 : 0;       // dS of a stage [128 keys][64 queries]
  // Q stages | dO stages | statistics | (fused: K tile | two dS tiles)
  __shared__ __attribute__((aligned(1024))) char smem[kPlainBytes + kKeyTileBytes + 2 * kDsBytes];
  char* const key_tile = smem + kPlainBytes;
  char* const ds_tiles = key_tile + kKeyTileBytes;

  // the workgroups behind the units sum the dQ partials that the dQ kernel left
  if (!FUSED && (int)blockIdx.x >= unit_blocks) {
    dq_tile_combine<D>(blockIdx.x - unit_blocks, hdr, max_items, row_items, row_partials, dq, Hq, scale, smem);
    return;
  }
  int unit_idx, head;
  decode_block(blockIdx.x, Hq, unit_idx, head);
  // both loads in flight together; the unit array always has max_units >= grid / Hq entries
  const int n_units = hdr->n_col_units;
  varlen_attn_unit it = units[min(unit_idx, max_units - 1)];
  // Grouped-query attention on large microbatches: a unit sweeps `hpu` q heads of its group
  // one after the other (dK, dV add up in the registers).  The workgroup ids are then decoded
  // for Hq / hpu head groups, so that the working ones still spread over all XCDs, and the
  // unit is fetched again (one more round trip in front of a long unit).
  const int hpu = hdr->col_heads_per_unit;
  if (hpu > 1) {
    decode_block(blockIdx.x, Hq / hpu, unit_idx, head);
    head *= hpu;
    it = units[min(unit_idx, max_units - 1)];
  }
  if (unit_idx >= n_units) return;
  const int kvh = head / (Hq / Hkv);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, c = lane & 31;
  const float cs = folded_scale(scale) * kLog2e;

  // from the thread index, not from the scalar `wave`: the branches between the two forms of a stage
  // then stay exec-masked, one behind the other, and the accumulators keep their registers; as scalar
  // branches the register allocator copies up to 270 of them per stage and spills
  const int wave_kv0 = it.row0 + 32 * (tid >> 6);
  const int my_kv = wave_kv0 + c;
  const bool kv_valid = my_kv < it.doc_end;
  const bool wave_active = wave_kv0 < it.doc_end;
  const int n_steps = it.step_end - it.step_begin;

  const __bf16* qbase = q + (size_t)head * D;
  const __bf16* dobase = d_o + (size_t)head * D;
  const float* lse_h = neg_lse + (size_t)head * N;
  const float* dsum_h = neg_dsum + (size_t)head * N;
  float* dq_acc_h = FUSED ? dq_acc + (size_t)head * D : nullptr;
  int heads_left = hpu;
  // this wave's share of the stages, and its statistics: wave w loads -LSE / scale (w even) or -D (w odd)
  // into the copy of its pair and reads both from that copy
  const unsigned lds_q = lds_addr_of(smem) + wave * 1024, lds_do = lds_q + NS * kStageBytes;
  const unsigned lds_stat = lds_addr_of(smem) + 2 * NS * kStageBytes + (wave >> 1) * kStatBytes + (wave & 1) * 256;
  const char* stat_base = smem + 2 * NS * kStageBytes + (wave >> 1) * kStatBytes;

  // stages are requested in order, one per step, while the stage before them is computed: the
  // wave-uniform addresses of the next stage's first rows live in scalar registers
  Stream stream;
  stream.init(wave, lane, (unsigned)((size_t)Hq * D * 2));
  unsigned long long stat_next = 0;
  unsigned stat_voff = 0;
  auto aim = [&](int st) __attribute__((always_inline)) {   // at step st of the chain
    const int q0 = it.row0 + kStep * (it.step_begin + st);
    stream.aim(q0, it.doc_end - 1);
    if (q0 + kStep > it.doc_end) stat_voff = (unsigned)min(lane, it.doc_end - 1 - q0) * 4;
  };
  auto restart = [&]() __attribute__((always_inline)) {   // at the first step of a chain (of every head the unit sweeps)
    const int q0 = it.row0 + kStep * it.step_begin;
    const size_t first = (size_t)q0 * ((size_t)Hq * D * 2);
    stream.start(reinterpret_cast<const char*>(qbase) + first, reinterpret_cast<const char*>(dobase) + first);
    stat_next = uniform64((wave & 1 ? dsum_h : lse_h) + q0);
    stat_voff = lane * 4;
    aim(0);
  };
  // piece P of the next stage into LDS stage ST; the first piece brings the statistics along
  auto piece = [&](auto piece_c, auto stage_c) __attribute__((always_inline)) {
    constexpr int P = decltype(piece_c)::value, ST = decltype(stage_c)::value;
    stream.template piece<P>(lds_q + ST * kStageBytes, lds_do + ST * kStageBytes);
    if (P == 0) dma4(stat_next, stat_voff, lds_stat + ST * 2 * kStatBytes);
  };
  auto all_pieces = [&](auto stage_c) __attribute__((always_inline)) {
    static_for<KK>([&](auto p) __attribute__((always_inline)) { piece(p, stage_c); });
  };
  bf16x8 kf[KK], vf[KK];
  const size_t kv_off = ((size_t)min(my_kv, it.doc_end - 1) * Hkv + kvh) * D;
  load_row_frags<D>(k + kv_off, h, kf);
  load_row_frags<D>(v + kv_off, h, vf);
  if (__builtin_expect(score_fold(scale) != 1.0f, 0)) {   // out of line: jumping over it took 0.3 us
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int e = 0; e < 8; ++e) kf[kk][e] = (__bf16)((float)kf[kk][e] * score_fold(scale));
  }
  if (FUSED && !kv_valid) {   // rows past the document end must not enter dQ; elsewhere they are never stored
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) kf[kk] = vf[kk] = __builtin_bit_cast(bf16x8, uint4{0, 0, 0, 0});
  }
  FragOffsets<D> fo;
  fo.init(lane);
  if (FUSED) {
    StageLoader<D, kTile> key_loader;
    key_loader.init(wave, lane, (unsigned)((size_t)Hkv * D * 2));
    key_loader.issue(k + (size_t)kvh * D, it.row0, it.doc_end - 1, lds_addr_of(key_tile), wave);
  }
  wait_all_vm_visible();
  pin_frags(kf);
  pin_frags(vf);
  // this lane's row of the dS tiles: key 32 wave + c; element (key, query) sits in the 16-byte
  // chunk query / 8 of that row, swizzled like every tile
  // dS of one 32-query block, accumulator registers 8 cc .. 8 cc + 7 (queries 32 qb + 16 cc +
  // 4h + {0..3} and + 8), into the dS tile
  auto ds_store = [&](char* tile, const bf16x8& v, int qb, int cc) __attribute__((always_inline)) {
    const uint4 w = __builtin_bit_cast(uint4, v);
    const int ds_row_swz = swz<kStep>(32 * wave + c);     // recomputed: nothing extra stays live across a stage
    char* row = tile + (32 * wave + c) * (kStep * 2) + 8 * h;
    *reinterpret_cast<uint2*>(row + (((4 * qb + 2 * cc) ^ ds_row_swz) << 4)) = uint2{w.x, w.y};
    *reinterpret_cast<uint2*>(row + (((4 * qb + 2 * cc + 1) ^ ds_row_swz) << 4)) = uint2{w.z, w.w};
  };
  // dQ of one finished stage: this wave's 32 columns of the head dimension, all 64 queries,
  // summed over the key slices that hold a key some query of the stage may see
  auto dq_flush = [&](const char* tile, int q0) __attribute__((always_inline)) {
    const int keys = min(it.doc_end, q0 + kStep) - it.row0;
    const int cc_end = min(max((keys + 15) / 16, 0), kTile / 16);
    FragOffsets<kStep> fo_ds;      // the dS tile has rows of kStep elements
    fo_ds.init(lane);
    // the 2 x D / 32 blocks of 32 queries x 32 columns are dealt to the four waves
    constexpr int kBlocks = DB / 2;                      // per wave: 2 (D = 128), 1 (D = 64)
    const int db = DB == 4 ? wave : wave & 1;            // column block
    const int qb0 = DB == 4 ? 0 : wave >> 1;             // first (only) query block
    f32x16 acc[kBlocks];
#pragma unroll
    for (int b = 0; b < kBlocks; ++b) acc[b] = f32x16(0.f);
#pragma unroll 1
    for (int cc = 0; cc < cc_end; ++cc) {
      const bf16x8 kb = read_trans<D>(key_tile, fo, cc, db);
#pragma unroll
      for (int b = 0; b < kBlocks; ++b) {
        // offsets of query block qb0 + b (selected, not indexed: the table stays in registers)
        const int lo = (qb0 + b) ? fo_ds.trans[1][0] : fo_ds.trans[0][0];
        const int hi = (qb0 + b) ? fo_ds.trans[1][1] : fo_ds.trans[0][1];
        acc[b] = mfma(lds_read_tr8(tile + lo + cc * 16 * kStep * 2, tile + hi + cc * 16 * kStep * 2), kb, acc[b]);
      }
    }
    // (the 32 offsets are formed here every time: kept across the stages they are spilled, one load from scratch memory in
    // front of each atomic)
    size_t stride = (size_t)Hq * D;
    asm volatile("" : "+s"(stride));
    const int row0 = q0 + 32 * qb0 + 4 * h;
    float* const first = dq_acc_h + 32 * db + c + row0 * stride;
#pragma unroll
    for (int b = 0; b < kBlocks; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int i = 32 * b + 8 * (r / 4) + r % 4;
        if (row0 + i < it.doc_end) unsafeAtomicAdd(first + i * stride, acc[b][r]);
      }
  };

  f32x16 dkacc[DB], dvacc[DB], dvacc_upper[HALVES ? DB : 1];
#pragma unroll
  for (int i = 0; i < DB; ++i) { dkacc[i] = f32x16(0.f); dvacc[i] = f32x16(0.f); if (HALVES) dvacc_upper[i] = f32x16(0.f); }

  // A 64-query stage against this wave's 32 keys: the two 32-query blocks are software-pipelined
  // by hand (this kernel runs one wave per SIMD, so nothing else hides LDS latency or overlaps
  // the exponentials with the matrix pipe):
  //   R0 | M1(0) + R1 | V(0) with M1(1) + T0 | M2(0) with V(1) + T1 | M2(1)
  // R: row-fragment and statistics reads, T: transposed-fragment reads, M1: S and dP,
  // V: P and dS on the vector ALU, M2: dV and dK.  Each matrix instruction is written next to
  // the vector and LDS work that should ride on it, and the fences keep that order.
  // MASKED: the stage touches the diagonal or runs past the document end (queries there are
  // clamped duplicates): P of a (query, key) pair outside the mask is set to exactly 0.
  // The direct-to-LDS loads of the next stage are issued one by one in M1(0), the phase with the
  // fewest other instructions per matrix instruction.
  auto stage = [&](const char* qt, const char* dot, const char* st, int q0, char* ds_tile, auto next_c, auto masked_c)
      __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    bf16x8 qa[KK], da[KK], qb[KK], db_[KK];
    bf16x8 tq0[2][DB], td0[2][DB], tq1[2][DB], td1[2][DB];
    bf16x8 pb0[2], dsb0[2], pb1[2], dsb1[2];
    f32x16 s0, s1, dp0, dp1;
    // softmax of element r of one block: p = exp(scale s - lse), ds = p (dp - D).  The matrix
    // instructions of S start from -lse / scale and those of dP from -D (both read from LDS straight
    // into the accumulators), so that no subtraction is left and no register holds the statistics
    // (r stands for query q0 + 32 qb + 8 (r / 4) + 4 h + r % 4)
    const int t_lo = my_kv - q0 - 4 * h, t_hi = it.doc_end - q0 - 4 * h;   // allowed: t_lo <= 32 qb + 8 (r / 4) + r % 4 < t_hi
    auto soft = [&](f32x16& sv, const f32x16& dpv, bf16x8 (&pb)[2], bf16x8 (&dsb)[2], int r, int qb)
        __attribute__((always_inline)) {
      float e = __builtin_amdgcn_exp2f(sv[r] * cs);
      if (MASKED) {
        const int t = 32 * qb + 8 * (r >> 2) + (r & 3);
        if (t < t_lo || t >= t_hi) e = 0.f;
      }
      sv[r] = e;
      if (r & 1) {   // the pair r - 1, r as bf16
        const f32x2 p = {sv[r - 1], e}, ds = {sv[r - 1] * dpv[r - 1], e * dpv[r]};
        const bf16x2 p2 = __builtin_convertvector(p, bf16x2), ds2 = __builtin_convertvector(ds, bf16x2);
#pragma unroll
        for (int i = 0; i < 2; ++i) { pb[r >> 3][(r & 7) - 1 + i] = p2[i]; dsb[r >> 3][(r & 7) - 1 + i] = ds2[i]; }
      }
    };
    // elements of the softmax beside matrix instruction i of 2 KK: none beside the first SKEW (their
    // scores are still in the matrix pipe), the rest evenly
    auto soft_slot = [&](f32x16& sv, const f32x16& dpv, bf16x8 (&pb)[2], bf16x8 (&dsb)[2], auto i_c, int qb)
        __attribute__((always_inline)) {
      constexpr int i = decltype(i_c)::value;
      constexpr int slots = 2 * KK - SKEW;
      constexpr int first = i < SKEW ? 0 : 16 * (i - SKEW) / slots, last = i < SKEW ? 0 : 16 * (i + 1 - SKEW) / slots;
#pragma unroll
      for (int e = first; e < last; ++e) soft(sv, dpv, pb, dsb, e, qb);
    };
    // ---- R0
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) {
      set4(s0, rq, *reinterpret_cast<const f32x4*>(st + (8 * rq + 4 * h) * 4));
      set4(dp0, rq, *reinterpret_cast<const f32x4*>(st + 256 + (8 * rq + 4 * h) * 4));
    }
    __builtin_amdgcn_sched_barrier(0);
    static_for<KK>([&](auto kk) __attribute__((always_inline)) {
      qa[kk] = lds_read_frag(qt, fo.row_frag[kk]);
      da[kk] = lds_read_frag(dot, fo.row_frag[kk]);
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- M1(0) + R1
    static_for<KK>([&](auto kk_c) {
      constexpr int kk = decltype(kk_c)::value;
      mfma_s(s0, qa[kk], kf[kk]);
      qb[kk] = lds_read_frag(qt, fo.row_frag[kk] + 32 * D * 2);
      if (kk < 4) set4(s1, kk, *reinterpret_cast<const f32x4*>(st + (32 + 8 * kk + 4 * h) * 4));
      __builtin_amdgcn_sched_barrier(0);
      piece(kk_c, next_c);
      __builtin_amdgcn_sched_barrier(0);
      mfma_s(dp0, da[kk], vf[kk]);
      db_[kk] = lds_read_frag(dot, fo.row_frag[kk] + 32 * D * 2);
      if (kk < 4) set4(dp1, kk, *reinterpret_cast<const f32x4*>(st + 256 + (32 + 8 * kk + 4 * h) * 4));
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- V(0) with M1(1) + T0
    static_for<KK>([&](auto kk_c) {
      constexpr int kk = decltype(kk_c)::value;
      mfma_s(s1, qb[kk], kf[kk]);
      soft_slot(s0, dp0, pb0, dsb0, std::integral_constant<int, 2 * kk>{}, 0);
      td0[kk / DB][kk % DB] = read_trans<D>(dot, fo, kk / DB, kk % DB);
      __builtin_amdgcn_sched_barrier(0);
      mfma_s(dp1, db_[kk], vf[kk]);
      soft_slot(s0, dp0, pb0, dsb0, std::integral_constant<int, 2 * kk + 1>{}, 0);
      tq0[kk / DB][kk % DB] = read_trans<D>(qt, fo, kk / DB, kk % DB);
      if (FUSED && (kk == KK / 2 - 1 || kk == KK - 1)) ds_store(ds_tile, dsb0[kk == KK - 1], 0, kk == KK - 1);
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- M2(0) with V(1) + T1
    static_for<2 * DB>([&](auto j_c) {
      constexpr int j = decltype(j_c)::value;
      dvacc[j % DB] = mfma(td0[j / DB][j % DB], pb0[j / DB], dvacc[j % DB]);
      soft_slot(s1, dp1, pb1, dsb1, std::integral_constant<int, 2 * j>{}, 1);
      td1[j / DB][j % DB] = read_trans<D>(dot + 32 * D * 2, fo, j / DB, j % DB);
      __builtin_amdgcn_sched_barrier(0);
      dkacc[j % DB] = mfma(tq0[j / DB][j % DB], dsb0[j / DB], dkacc[j % DB]);
      soft_slot(s1, dp1, pb1, dsb1, std::integral_constant<int, 2 * j + 1>{}, 1);
      tq1[j / DB][j % DB] = read_trans<D>(qt + 32 * D * 2, fo, j / DB, j % DB);
      if (FUSED && (j == KK / 2 - 1 || j == KK - 1)) ds_store(ds_tile, dsb1[j == KK - 1], 1, j == KK - 1);
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- M2(1)
#pragma unroll
    for (int cc = 0; cc < 2; ++cc)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        if constexpr (HALVES) dvacc_upper[db] = mfma(td1[cc][db], pb1[cc], dvacc_upper[db]);
        else dvacc[db] = mfma(td1[cc][db], pb1[cc], dvacc[db]);
        dkacc[db] = mfma(tq1[cc][db], dsb1[cc], dkacc[db]);
      }
  };
  auto body = [&](int st, auto stage_c) {
    constexpr int ST = decltype(stage_c)::value;
    const std::integral_constant<int, 1 - ST> next_c{};
    wait_vm<0>();
    __syncthreads();
    // the last step requests its own stage again (into the other buffer; nobody reads it), so that
    // every step is the same
    if (st < n_steps - 1) {
      stream.advance();
      stat_next += kStep * 4;
      aim(st + 1);
    }
    const int step = it.step_begin + st;
    const int q0 = it.row0 + kStep * step;
    // fused: dQ of the previous stage, whose dS every wave has written before the barrier above
    if (FUSED && st > 0) dq_flush(ds_tiles + (1 - ST) * kDsBytes, q0 - kStep);
    // no keys, or every query of the stage lies before this wave's keys
    if (!wave_active || q0 + kStep - 1 < wave_kv0) { all_pieces(next_c); return; }
    const char* qt = smem + ST * kStageBytes;
    const char* dot = smem + (NS + ST) * kStageBytes;
    const char* stt = stat_base + ST * 2 * kStatBytes;
    char* ds_tile = ds_tiles + ST * kDsBytes;
    if (q0 < wave_kv0 + 32 || q0 + kStep > it.doc_end) stage(qt, dot, stt, q0, ds_tile, next_c, std::true_type{});
    else stage(qt, dot, stt, q0, ds_tile, next_c, std::false_type{});
  };
  for (;;) {
    restart();
    all_pieces(std::integral_constant<int, 0>{});
    for (int st = 0; st < n_steps; st += NS) {
      body(st, std::integral_constant<int, 0>{});
      if (st + 1 >= n_steps) break;
      body(st + 1, std::integral_constant<int, 1>{});
    }
    wait_vm<0>();  // nothing may still be landing in LDS when the workgroup goes on or retires
    if (FUSED) {       // dQ of the chain's last stage
      __syncthreads();
      dq_flush(ds_tiles + ((n_steps - 1) & 1) * kDsBytes, it.row0 + kStep * (it.step_begin + n_steps - 1));
    }
    if (--heads_left == 0) break;
    __syncthreads();   // every wave is done with the stages before they are refilled
    qbase += D; dobase += D; lse_h += N; dsum_h += N;
    if (FUSED) dq_acc_h += D;
  }

  if constexpr (HALVES)
#pragma unroll
    for (int i = 0; i < DB; ++i) dvacc[i] += dvacc_upper[i];
  if (it.slot >= 0) {
    float* part = partials + ((size_t)it.slot * Hq + head) * 2 * frag_floats<D>();
    store_frag<D>(part, dkacc, wave, lane);
    store_frag<D>(part + frag_floats<D>(), dvacc, wave, lane);
    return;
  }
  __syncthreads();   // every wave is done with the stages
  {
    char* tile = smem + 2 * wave * RowTile<D>::kBytes;
    const size_t first = ((size_t)wave_kv0 * Hkv + kvh) * D;
    store_rows<D>(tile, dk + first, (size_t)Hkv * D, it.doc_end - wave_kv0, dkacc, lane, scale);
    store_rows<D>(tile + RowTile<D>::kBytes, dv + first, (size_t)Hkv * D, it.doc_end - wave_kv0, dvacc, lane, 1.0f);
  }
}

// Adds up the [dK | dV] fp32 partial fragments of cut or grouped column tiles in a fixed order
// (chunks in chain order, then the q heads of the group) and stores bf16 rows; dK is multiplied by
// `scale`.  Elementwise, work dealt as in fwd_combine_kernel (two column blocks of one wave's rows
// of one tensor; up to four partials in flight; a fixed number of workgroups walks over the items).
// The dQ partials are summed at the end of the dK/dV kernel's grid.
template <int D>
__global__ void __launch_bounds__(kThreads)
bwd_combine_kernel(const varlen_attn_plan_header* __restrict__ hdr,
                   const varlen_attn_combine_item* __restrict__ items, int max_items,
                   const float* __restrict__ partials, __bf16* __restrict__ dk,
                   __bf16* __restrict__ dv, int Hq, int Hkv, float scale) {
  constexpr int DB = D / 32;
  constexpr int kPieces = 2 * 4 * DB / 2;   // of an (item, kv head): dK and dV, 4 waves, pairs of column blocks
  constexpr int kFlight = 4;
  constexpr size_t psize = 2 * frag_floats<D>();
  using Tile = RowTile<64>;
  __shared__ __attribute__((aligned(16))) char tiles[2][Tile::kBytes];
  int buf = 0;   // two tiles in turn: one barrier per item
  const int lane = threadIdx.x & 63, rq = threadIdx.x >> 6, h = lane >> 5, c = lane & 31;
  const int n_items = hdr->n_col_combine, hpu = hdr->col_heads_per_unit;
  const int G = Hq / Hkv;
  for (int work = blockIdx.x; work < max_items * Hkv * kPieces; work += gridDim.x) {
    const int piece = work % kPieces, rest = work / kPieces;
    const int idx = rest / Hkv, oh = rest % Hkv;
    const varlen_attn_combine_item it = items[idx];   // in flight together with n_items
    if (idx >= n_items) return;
    const int tensor = piece & 1, wave = (piece >> 1) / (DB / 2), db = 2 * ((piece >> 1) % (DB / 2));
    const int row0 = it.row0 + 32 * wave;
    if (row0 >= it.doc_end) continue;   // (rows past the end inside the block: computed, not stored)
    const float* p0 = partials + ((size_t)it.slot0 * Hq + oh * G) * psize + tensor * frag_floats<D>() +
                      (size_t)(wave * DB + db) * kThreads * 4 + (size_t)threadIdx.x * 4;
    // of the G heads of a group only every hpu-th holds a partial (its unit swept hpu heads);
    // partial number j = ch * Gp + g sits (ch * Hq + g * hpu) partial sizes after the first
    const int Gp = G / hpu, n_parts = it.n_chunks * Gp;
    f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
#pragma unroll 1
    for (int j0 = 0; j0 < n_parts; j0 += kFlight) {
      f32x4 xa[kFlight], xb[kFlight];
#pragma unroll
      for (int j = 0; j < kFlight; ++j) {
        xa[j] = xb[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (j0 + j < n_parts) {   // the same for the whole workgroup
          const size_t off = ((size_t)((j0 + j) / Gp) * Hq + ((j0 + j) % Gp) * hpu) * psize;
          xa[j] = *reinterpret_cast<const f32x4*>(p0 + off);
          xb[j] = *reinterpret_cast<const f32x4*>(p0 + off + kThreads * 4);
        }
      }
#pragma unroll
      for (int j = 0; j < kFlight; ++j) { acc0 += xa[j]; acc1 += xb[j]; }
    }
    const float mul = tensor == 0 ? scale : 1.0f;
    Tile::put(tiles[buf], c, h, rq, pack4(acc0[0] * mul, acc0[1] * mul, acc0[2] * mul, acc0[3] * mul));
    Tile::put(tiles[buf], c, h, 4 + rq, pack4(acc1[0] * mul, acc1[1] * mul, acc1[2] * mul, acc1[3] * mul));
    __syncthreads();
    const int out_row = row0 + (threadIdx.x >> 3), chunk = threadIdx.x & 7;
    const uint4 w = Tile::get(tiles[buf], threadIdx.x >> 3, chunk);
    if (out_row < it.doc_end)
      *reinterpret_cast<uint4*>((tensor == 0 ? dk : dv) + ((size_t)out_row * Hkv + oh) * D + 32 * db + 8 * chunk) = w;
    buf ^= 1;
  }
}

}  // namespace

#endif  // VARLEN_ATTN_BWD_HPP_
