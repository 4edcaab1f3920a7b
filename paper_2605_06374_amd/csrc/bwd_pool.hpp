// Backward as one pool of work: dQ units and dK/dV units drawn by resident workgroups.
#ifndef VARLEN_ATTN_BWD_POOL_HPP_
#define VARLEN_ATTN_BWD_POOL_HPP_

#include "tiles.hpp"
#include "staging.hpp"
#include "fragments.hpp"
#include "plan.hpp"

namespace {

// ----------------------------------------------------------------------------------------
// Backward with heads of 128 (the rule: pooled_backward() in varlen_attn.hip).  One workgroup per compute unit stays and draws
// units, column units (dK, dV) first, then units of dQ, longest first within each: the short dQ units fill what
// the column units leave idle, where a kernel each has a tail, a burst of first loads and a launch of its own.  dQ has
// units of its own (plan.hpp): in the pool a chain needs no cut until it would outlast the rest, which leaves a
// quarter of the partial results at 8192 tokens.  Nothing depends on the order in which units are drawn, so that the
// results are reproducible.  The price is D: both kinds need it, so it comes from a pass in front (bwd_prep_kernel).
//
// What bounds it: at 512 registers one wave per SIMD issues everything, and on large microbatches the clock, which the
// power limit takes down to 1.7 - 2.0 GHz on real operands (2.2 on zeros; cycles of a die over the launch's duration).  The matrix
// pipe is busy in 0.33 of these cycles at 8192 tokens in 9 documents, 0.50 at 32768 in 35 and 0.62 at 32768 in 11.  Both sweeps
// are therefore pipelined by hand: the streamed rows come in stages of 64, two blocks of 32 of which
//   M1(0) + R1 | V(0) with M1(1) + T0 | M2(0) with V(1) + T1 | wait, barrier | M2(1) + R0 of the next stage
// (R: row fragments and statistics from LDS, T: transposed fragments, M1: S and dP, V: P and dS on the vector ALU, M2: the
// sums).  The barrier lies in front of M2(1), whose operands are in registers by then, so that the first reads of the next
// stage run behind its matrix instructions and no wave meets an empty matrix pipe behind the barrier (all kernels of
// a backward at 32768 tokens in 11 documents 1235 -> 1196 us).  The stationary fragments live in accumulation
// registers, which the matrix instructions read as well: with them in vector registers the read-ahead spilled.
// Two kernels and their reduction / statistics pass, pool and reduction, us of a whole step: 117 / 107 at 8192 tokens in 9
// documents, 48.4 / 42.5 at 4096 in 61, 629 / 604 at 16384 with 8 q heads on one kv head, 1674 / 1631 at 32768 in 11.
// Measured and left out: row units first, which publish D themselves, with a wait in front of the column units (loads
// past the L2 and 250 increments of one counter: 44 instead of 23 us at 4096 tokens); the next unit's stationary
// tiles through LDS while the last stages run (its bookkeeping costs each of those stages as much as the
// loads would); a wait that leaves a unit's stores behind (no difference).
// ----------------------------------------------------------------------------------------

// The results of S and dP are not touched until two further matrix instructions have been issued (tiles.hpp)
constexpr int kSkew = 2;

// S and dP: accumulators in vector registers, the stationary operand in accumulation registers
__device__ __forceinline__ void mfma_vgpr_agpr(f32x16& c, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "a"(b));
}
// ... the first of a sum, from a constant accumulator (a statistic of the lane's row in every register)
__device__ __forceinline__ void mfma_vgpr_from(f32x16& c, const bf16x8& a, const bf16x8& b, const f32x16& init) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(c) : "v"(a), "a"(b), "v"(init));
}
template <int KK>
__device__ __forceinline__ void pin_frags_acc(bf16x8 (&f)[KK]) {
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) asm volatile("" : "+a"(f[kk]));
}

// The units of a pool are dealt by tickets, column units first, one counter per group of heads (the heads whose K, V, Q
// and dO lines share the L2 of the group's XCDs).  A workgroup's first ticket is its own number in its group, later
// ones come from the counter.
struct TicketGroup {
  int index, heads, stride, members, first;   // counter; head groups per unit number; workgroups of the group; own number
  int hpu, n_col, total;
  __device__ __forceinline__ void init(int bid, int groups, int Hq, int hpu_, int n_col_, int n_row) {
    hpu = hpu_;
    const int Hv = Hq / hpu, xcd = bid % 8;
    if (8 % Hv == 0) { index = xcd % Hv; heads = 1; first = (bid / 8) * (8 / Hv) + xcd / Hv; members = groups / Hv; }
    else if (Hv % 8 == 0) { index = xcd; heads = Hv / 8; first = bid / 8; members = groups / 8; }
    else { index = 0; heads = Hv; first = bid; members = groups; }
    stride = Hv % 8 == 0 ? 8 : 1;
    n_col = n_col_ * heads;
    total = n_col + n_row * heads * hpu;
  }
  __device__ __forceinline__ void decode(int t, int& unit, int& head) const {
    if (t < n_col) {
      unit = heads == 1 ? t : __builtin_amdgcn_readfirstlane(t / heads);
      head = (index + stride * (t - unit * heads)) * hpu;
    } else {
      const int r = t - n_col, per = heads * hpu;
      unit = per == 1 ? r : __builtin_amdgcn_readfirstlane(r / per);
      const int j = r - unit * per, v = hpu == 1 ? j : __builtin_amdgcn_readfirstlane(j / hpu);
      head = (index + stride * v) * hpu + (j - v * hpu);
    }
  }
};

// The next ticket: thread 0 asks for it in front of a unit's last stage but one and passes it on through LDS in front of
// the last, whose barrier publishes it.  (Units of one stage: in front of that, both.)
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
    __syncthreads();   // (the last stage's read-ahead ends)
    return __builtin_amdgcn_readfirstlane(*lds);
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
  int N, Hq, Hkv;
  float scale;
  int* tickets;
};

// LDS of a workgroup: two stages of two streamed tiles (K and V, or Q and dO), then the statistics of the streamed queries:
// -LSE / scale [64], -D [64] per stage, two copies, one per pair of waves
template <int D>
struct BwdLds {
  static constexpr int kStage = kStep * D * 2, kStat = 512;
  static constexpr int kStats = 4 * kStage, kBytes = kStats + 4 * kStat;
};

// The units are objects: open() sends the loads of a unit's first stage and of its stationary rows on their way, sweep()
// walks its chain, store() writes the results.  The next unit is opened before the results of the last one are stored.
template <int D>
struct DqUnit {
  static constexpr int KK = D / 16, DB = D / 32, NS = 2, kStage = BwdLds<D>::kStage;
  varlen_attn_unit it;
  int head;
  PairStream<D, kStep> stream;
  bf16x8 qf[KK], dof[KK];
  float neg_lse_row, neg_dsum_row;

  __device__ __forceinline__ void open(const BwdArgs<D>& a, const varlen_attn_unit& unit, int head_, char* smem) {
    it = unit;
    head = head_;
    const int Hq = a.Hq, Hkv = a.Hkv, kvh = head / (Hq / Hkv);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kv_first = it.doc_start + kStep * it.step_begin;
    stream.init(wave, lane, (unsigned)((size_t)Hkv * D * 2));
    stream.start(a.k + ((size_t)kv_first * Hkv + kvh) * D, a.v + ((size_t)kv_first * Hkv + kvh) * D);
    stream.aim(kv_first, it.doc_end - 1);
    const unsigned lds_k = lds_addr_of(smem) + wave * 1024;
    static_for<KK>([&](auto p) __attribute__((always_inline)) { stream.template piece<decltype(p)::value>(lds_k, lds_k + NS * kStage); });
    const int row = min(it.row0 + 32 * (tid >> 6) + (lane & 31), it.doc_end - 1);   // rows past the document end: duplicates, never stored
    const size_t row_off = ((size_t)row * Hq + head) * D;
    neg_lse_row = a.neg_lse[(size_t)head * a.N + row];
    neg_dsum_row = a.neg_dsum[(size_t)head * a.N + row];
    load_row_frags<D>(a.d_o + row_off, lane >> 5, dof);
    load_row_frags<D>(a.q + row_off, lane >> 5, qf);
  }

  // S^T = K Q^T, dP^T = V dO^T, dQ^T += K^T dS^T
  template <typename Tickets>
  __device__ __forceinline__ void sweep(const BwdArgs<D>& a, char* smem, const FragOffsets<D>& fo, f32x16 (&acc)[DB], Tickets& tickets) {
    auto mfma_s = [&](f32x16& c, const bf16x8& x, const bf16x8& y, const f32x16& init, auto first_c) __attribute__((always_inline)) {
      if constexpr (decltype(first_c)::value) mfma_vgpr_from(c, x, y, init);
      else mfma_vgpr_agpr(c, x, y);
    };
    const float scale = a.scale, cs = folded_scale(scale) * kLog2e;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, c = lane & 31;
    const int wave_row0 = it.row0 + 32 * (tid >> 6);
    const int my_row = wave_row0 + c;
    const bool wave_active = it.row0 + 32 * wave < it.doc_end;   // (a scalar branch)
    const int wave_last_row = min(it.row0 + 32 * wave + 31, it.doc_end - 1);
    const int n_steps = it.step_end - it.step_begin;
    const unsigned lds_k = lds_addr_of(smem) + wave * 1024, lds_v = lds_k + NS * kStage;
    const int kv_first = it.doc_start + kStep * it.step_begin;
    auto piece = [&](auto piece_c, auto stage_c) __attribute__((always_inline)) {
      constexpr int P = decltype(piece_c)::value, ST = decltype(stage_c)::value;
      stream.template piece<P>(lds_k + ST * kStage, lds_v + ST * kStage);
    };
    auto all_pieces = [&](auto stage_c) __attribute__((always_inline)) {
      static_for<KK>([&](auto p) __attribute__((always_inline)) { piece(p, stage_c); });
    };
    f32x16 s_init = f32x16(neg_lse_row), dp_init = f32x16(neg_dsum_row);
    if (__builtin_expect(score_fold(scale) != 1.0f, 0)) {
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[kk][e] = (__bf16)((float)qf[kk][e] * score_fold(scale));
  }
  pin_frags_acc(qf);
  pin_frags_acc(dof);
  asm volatile("" : "+v"(s_init), "+v"(dp_init));
#pragma unroll
  for (int i = 0; i < DB; ++i) acc[i] = f32x16(0.f);

  bf16x8 ka[KK], va[KK];
  auto stage = [&](int kv0, auto stage_c, auto masked_c) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    constexpr int ST = decltype(stage_c)::value;
    const char* kt = smem + ST * kStage;
    const char* vt = smem + (2 + ST) * kStage;
    bf16x8 kb[KK], vb[KK];
    bf16x8 tk0[2][DB], tk1[2][DB];
    bf16x8 dsb0[2], dsb1[2];
    f32x16 s0, s1, dp0, dp1;
    const int t_hi = my_row - kv0 - 4 * h;   // allowed: 32 block + 8 (r / 4) + r % 4 <= t_hi
    auto soft = [&](f32x16& sv, const f32x16& dpv, bf16x8 (&dsb)[2], int r, int kb_) __attribute__((always_inline)) {
      float e = __builtin_amdgcn_exp2f(sv[r] * cs);
      if (MASKED) {
        if (32 * kb_ + 8 * (r >> 2) + (r & 3) > t_hi) e = 0.f;
      }
      sv[r] = e * dpv[r];
      if (r & 1) {
        const f32x2 ds = {sv[r - 1], sv[r]};
        const bf16x2 ds2 = __builtin_convertvector(ds, bf16x2);
#pragma unroll
        for (int i = 0; i < 2; ++i) dsb[r >> 3][(r & 7) - 1 + i] = ds2[i];
      }
    };
    auto soft_slot = [&](f32x16& sv, const f32x16& dpv, bf16x8 (&dsb)[2], auto i_c, auto n_c, int kb_)
        __attribute__((always_inline)) {
      constexpr int i = decltype(i_c)::value, slots = decltype(n_c)::value - kSkew;
      constexpr int first = i < kSkew ? 0 : 16 * (i - kSkew) / slots, last = i < kSkew ? 0 : 16 * (i + 1 - kSkew) / slots;
#pragma unroll
      for (int e = first; e < last; ++e) soft(sv, dpv, dsb, e, kb_);
    };
    static_for<KK>([&](auto kk_c) {
      constexpr int kk = decltype(kk_c)::value;
      mfma_s(s0, ka[kk], qf[kk], s_init, std::bool_constant<kk == 0>{});
      kb[kk] = lds_read_frag(kt, fo.row_frag[kk] + 32 * D * 2);
      __builtin_amdgcn_sched_barrier(0);
      piece(kk_c, std::integral_constant<int, 1 - ST>{});
      __builtin_amdgcn_sched_barrier(0);
      mfma_s(dp0, va[kk], dof[kk], dp_init, std::bool_constant<kk == 0>{});
      vb[kk] = lds_read_frag(vt, fo.row_frag[kk] + 32 * D * 2);
      __builtin_amdgcn_sched_barrier(0);
    });
    static_for<KK>([&](auto kk_c) {
      constexpr int kk = decltype(kk_c)::value;
      mfma_s(s1, kb[kk], qf[kk], s_init, std::bool_constant<kk == 0>{});
      soft_slot(s0, dp0, dsb0, std::integral_constant<int, 2 * kk>{}, std::integral_constant<int, 2 * KK>{}, 0);
      tk0[kk / DB][kk % DB] = read_trans<D>(kt, fo, kk / DB, kk % DB);
      __builtin_amdgcn_sched_barrier(0);
      mfma_s(dp1, vb[kk], dof[kk], dp_init, std::bool_constant<kk == 0>{});
      soft_slot(s0, dp0, dsb0, std::integral_constant<int, 2 * kk + 1>{}, std::integral_constant<int, 2 * KK>{}, 0);
      __builtin_amdgcn_sched_barrier(0);
    });
    static_for<2 * DB>([&](auto j_c) {
      constexpr int j = decltype(j_c)::value;
      acc[j % DB] = mfma(tk0[j / DB][j % DB], dsb0[j / DB], acc[j % DB]);
      soft_slot(s1, dp1, dsb1, j_c, std::integral_constant<int, 2 * DB>{}, 1);
      tk1[j / DB][j % DB] = read_trans<D>(kt + 32 * D * 2, fo, j / DB, j % DB);
      __builtin_amdgcn_sched_barrier(0);
    });
    wait_vm<0>();
    __syncthreads();
    // A wave's only masked stage holds the diagonal, of an even wave in its first block: the second, above it, is left out, not
    // multiplied by zeros, so that an infinity or NaN in K or V reaches dQ of the 31 rows in front of its token at most, as in
    // bwd_dq_kernel.  (By the matrix instruction: with the whole phase left out packs of short documents take 1 % longer, and
    // with a stage of one block as a third form longer chains up to 2 %.)
    static_for<2 * DB>([&](auto j_c) {
      constexpr int j = decltype(j_c)::value;
      if (!MASKED || (wave & 1)) acc[j % DB] = mfma(tk1[j / DB][j % DB], dsb1[j / DB], acc[j % DB]);
      ka[j] = lds_read_frag(smem + (1 - ST) * kStage, fo.row_frag[j]);
      va[j] = lds_read_frag(smem + (3 - ST) * kStage, fo.row_frag[j]);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // steps that hold a key for this wave: all but the last ones of the diagonal (none where the chunk begins behind its rows)
  const int my_steps = wave_active ? min(n_steps, (wave_last_row - kv_first + kStep) / kStep) : 0;
  int st = 0;
  if (n_steps == 1) tickets.step(0);
  auto to_next = [&]() __attribute__((always_inline)) {   // the last step requests its own stage again (nobody reads it)
    const int kv0 = kv_first + kStep * st;
    if (++st < n_steps) {
      stream.advance();
      stream.aim(kv0 + kStep, it.doc_end - 1);
    }
    if (st >= n_steps - 1) tickets.step(st - (n_steps - 1));
    return kv0;
  };
  auto body = [&](auto stage_c) __attribute__((always_inline)) {
    const int kv0 = to_next();
    if (kv0 + kStep - 1 > wave_row0) stage(kv0, stage_c, std::true_type{});
    else stage(kv0, stage_c, std::false_type{});
  };
  __syncthreads();
  if (my_steps > 0) {
    static_for<KK>([&](auto kk) __attribute__((always_inline)) {
      ka[kk] = lds_read_frag(smem, fo.row_frag[kk]);
      va[kk] = lds_read_frag(smem + NS * kStage, fo.row_frag[kk]);
    });
    for (;;) {
      body(std::integral_constant<int, 0>{});
      if (st >= my_steps) break;
      body(std::integral_constant<int, 1>{});
      if (st >= my_steps) break;
    }
  }
  while (st < n_steps) {
    to_next();
    if (st & 1) all_pieces(std::integral_constant<int, 1>{});
    else all_pieces(std::integral_constant<int, 0>{});
    wait_vm<0>();
    __syncthreads();
  }
  }
};

template <int D>
__device__ __forceinline__ void store_dq(const BwdArgs<D>& a, const varlen_attn_unit& it, int head, char* tile, const f32x16 (&acc)[D / 32]) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (it.slot >= 0)
    store_frag<D>(a.row_partials + ((size_t)it.slot * a.Hq + head) * frag_floats<D>(), acc, wave, lane);
  else
    store_rows<D>(tile, a.dq + ((size_t)(it.row0 + 32 * wave) * a.Hq + head) * D, (size_t)a.Hq * D, it.doc_end - it.row0 - 32 * wave,
                  acc, lane, a.scale);
}

template <int D>
struct DkvUnit {
  static constexpr int KK = D / 16, DB = D / 32, NS = 2, kStage = BwdLds<D>::kStage, kStat = BwdLds<D>::kStat;
  varlen_attn_unit it;
  int head;            // the first of the `hpu` q heads of a group that the unit sweeps one after the other
  PairStream<D, kStep> stream;
  unsigned long long stat_next;
  unsigned stat_voff;
  bf16x8 kf[KK], vf[KK];

  __device__ __forceinline__ void aim(int q0) {
    stream.aim(q0, it.doc_end - 1);
    if (q0 + kStep > it.doc_end) stat_voff = (unsigned)min((int)(threadIdx.x & 63), it.doc_end - 1 - q0) * 4;
  }
  __device__ __forceinline__ void start(const BwdArgs<D>& a, int h, int wave) {   // at the first step of the chain, q head h
    const int q0 = it.row0 + kStep * it.step_begin;
    const size_t first = ((size_t)q0 * a.Hq + h) * D;
    stream.start(a.q + first, a.d_o + first);
    stat_next = uniform64((wave & 1 ? a.neg_dsum : a.neg_lse) + (size_t)h * a.N + q0);
    stat_voff = (threadIdx.x & 63) * 4;
    aim(q0);
  }
  template <int P, int ST>
  __device__ __forceinline__ void piece(unsigned lds, int wave) const {
    stream.template piece<P>(lds + wave * 1024 + ST * kStage, lds + wave * 1024 + (NS + ST) * kStage);
    if (P == 0) dma4(stat_next, stat_voff, lds + BwdLds<D>::kStats + (wave >> 1) * kStat + (wave & 1) * 256 + ST * 2 * kStat);
  }
  template <int ST>
  __device__ __forceinline__ void all_pieces(unsigned lds, int wave) const {
    static_for<KK>([&](auto p) __attribute__((always_inline)) { piece<decltype(p)::value, ST>(lds, wave); });
  }
  __device__ __forceinline__ void open(const BwdArgs<D>& a, const varlen_attn_unit& unit, int head_, char* smem) {
    it = unit;
    head = head_;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    stream.init(wave, lane, (unsigned)((size_t)a.Hq * D * 2));
    start(a, head, wave);
    all_pieces<0>(lds_addr_of(smem), wave);
    const size_t kv_off = ((size_t)min(it.row0 + 32 * (tid >> 6) + (lane & 31), it.doc_end - 1) * a.Hkv + head / (a.Hq / a.Hkv)) * D;
    load_row_frags<D>(a.k + kv_off, lane >> 5, kf);
    load_row_frags<D>(a.v + kv_off, lane >> 5, vf);
  }

  // S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS
  template <typename Tickets>
  __device__ __forceinline__ void sweep(const BwdArgs<D>& a, int hpu, char* smem, const FragOffsets<D>& fo, f32x16 (&dkacc)[DB],
                                        f32x16 (&dvacc)[DB], Tickets& tickets) {
    const float scale = a.scale, cs = folded_scale(scale) * kLog2e;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, c = lane & 31;
    const int wave_kv0 = it.row0 + 32 * (tid >> 6);
    const int my_kv = wave_kv0 + c;
    const bool wave_active = it.row0 + 32 * wave < it.doc_end;   // (a scalar branch)
    const int n_steps = it.step_end - it.step_begin;
    const unsigned lds = lds_addr_of(smem);
    const char* const stat_base = smem + BwdLds<D>::kStats + (wave >> 1) * kStat;
    if (__builtin_expect(score_fold(scale) != 1.0f, 0)) {   // out of line: jumping over it took 0.3 us
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
#pragma unroll
        for (int e = 0; e < 8; ++e) kf[kk][e] = (__bf16)((float)kf[kk][e] * score_fold(scale));
  }
  pin_frags_acc(kf);
  pin_frags_acc(vf);
#pragma unroll
  for (int i = 0; i < DB; ++i) { dkacc[i] = f32x16(0.f); dvacc[i] = f32x16(0.f); }

  // read ahead of a stage, behind the last matrix phase of the stage before it
  bf16x8 qa[KK], da[KK];
  f32x16 s0, dp0;
  auto read_ahead_stats = [&](auto stage_c) __attribute__((always_inline)) {
    const char* st = stat_base + decltype(stage_c)::value * 2 * kStat;
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) {
      set4(s0, rq, *reinterpret_cast<const f32x4*>(st + (8 * rq + 4 * h) * 4));
      set4(dp0, rq, *reinterpret_cast<const f32x4*>(st + 256 + (8 * rq + 4 * h) * 4));
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto stage = [&](int q0, auto stage_c, auto masked_c) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    constexpr int ST = decltype(stage_c)::value;
    const char* qt = smem + ST * kStage;
    const char* dot = smem + (2 + ST) * kStage;
    const char* st = stat_base + ST * 2 * kStat;
    bf16x8 qb[KK], db_[KK];
    bf16x8 tq0[2][DB], td0[2][DB], tq1[2][DB], td1[2][DB];
    bf16x8 pb0[2], dsb0[2], pb1[2], dsb1[2];
    f32x16 s1, dp1;
    const int t_lo = my_kv - q0 - 4 * h, t_hi = it.doc_end - q0 - 4 * h;
    auto soft = [&](f32x16& sv, const f32x16& dpv, bf16x8 (&pb)[2], bf16x8 (&dsb)[2], int r, int qb_)
        __attribute__((always_inline)) {
      float e = __builtin_amdgcn_exp2f(sv[r] * cs);
      if (MASKED) {
        const int t = 32 * qb_ + 8 * (r >> 2) + (r & 3);
        if (t < t_lo || t >= t_hi) e = 0.f;
      }
      sv[r] = e;
      if (r & 1) {
        const f32x2 p = {sv[r - 1], e}, ds = {sv[r - 1] * dpv[r - 1], e * dpv[r]};
        const bf16x2 p2 = __builtin_convertvector(p, bf16x2), ds2 = __builtin_convertvector(ds, bf16x2);
#pragma unroll
        for (int i = 0; i < 2; ++i) { pb[r >> 3][(r & 7) - 1 + i] = p2[i]; dsb[r >> 3][(r & 7) - 1 + i] = ds2[i]; }
      }
    };
    auto soft_slot = [&](f32x16& sv, const f32x16& dpv, bf16x8 (&pb)[2], bf16x8 (&dsb)[2], auto i_c, int qb_)
        __attribute__((always_inline)) {
      constexpr int i = decltype(i_c)::value;
      constexpr int slots = 2 * KK - kSkew;
      constexpr int first = i < kSkew ? 0 : 16 * (i - kSkew) / slots, last = i < kSkew ? 0 : 16 * (i + 1 - kSkew) / slots;
#pragma unroll
      for (int e = first; e < last; ++e) soft(sv, dpv, pb, dsb, e, qb_);
    };
    static_for<KK>([&](auto kk_c) {
      constexpr int kk = decltype(kk_c)::value;
      mfma_vgpr_agpr(s0, qa[kk], kf[kk]);
      qb[kk] = lds_read_frag(qt, fo.row_frag[kk] + 32 * D * 2);
      if (kk < 4) set4(s1, kk, *reinterpret_cast<const f32x4*>(st + (32 + 8 * kk + 4 * h) * 4));
      __builtin_amdgcn_sched_barrier(0);
      this->template piece<kk, 1 - ST>(lds, wave);
      __builtin_amdgcn_sched_barrier(0);
      mfma_vgpr_agpr(dp0, da[kk], vf[kk]);
      db_[kk] = lds_read_frag(dot, fo.row_frag[kk] + 32 * D * 2);
      if (kk < 4) set4(dp1, kk, *reinterpret_cast<const f32x4*>(st + 256 + (32 + 8 * kk + 4 * h) * 4));
      __builtin_amdgcn_sched_barrier(0);
    });
    static_for<KK>([&](auto kk_c) {
      constexpr int kk = decltype(kk_c)::value;
      mfma_vgpr_agpr(s1, qb[kk], kf[kk]);
      soft_slot(s0, dp0, pb0, dsb0, std::integral_constant<int, 2 * kk>{}, 0);
      td0[kk / DB][kk % DB] = read_trans<D>(dot, fo, kk / DB, kk % DB);
      __builtin_amdgcn_sched_barrier(0);
      mfma_vgpr_agpr(dp1, db_[kk], vf[kk]);
      soft_slot(s0, dp0, pb0, dsb0, std::integral_constant<int, 2 * kk + 1>{}, 0);
      tq0[kk / DB][kk % DB] = read_trans<D>(qt, fo, kk / DB, kk % DB);
      __builtin_amdgcn_sched_barrier(0);
    });
    static_for<2 * DB>([&](auto j_c) {
      constexpr int j = decltype(j_c)::value;
      dvacc[j % DB] = mfma(td0[j / DB][j % DB], pb0[j / DB], dvacc[j % DB]);
      soft_slot(s1, dp1, pb1, dsb1, std::integral_constant<int, 2 * j>{}, 1);
      td1[j / DB][j % DB] = read_trans<D>(dot + 32 * D * 2, fo, j / DB, j % DB);
      __builtin_amdgcn_sched_barrier(0);
      dkacc[j % DB] = mfma(tq0[j / DB][j % DB], dsb0[j / DB], dkacc[j % DB]);
      soft_slot(s1, dp1, pb1, dsb1, std::integral_constant<int, 2 * j + 1>{}, 1);
      tq1[j / DB][j % DB] = read_trans<D>(qt + 32 * D * 2, fo, j / DB, j % DB);
      __builtin_amdgcn_sched_barrier(0);
    });
    wait_vm<0>();
    __syncthreads();
    read_ahead_stats(std::integral_constant<int, 1 - ST>{});
    static_for<2 * DB>([&](auto j_c) {
      constexpr int j = decltype(j_c)::value;
      dvacc[j % DB] = mfma(td1[j / DB][j % DB], pb1[j / DB], dvacc[j % DB]);
      qa[j] = lds_read_frag(smem + (1 - ST) * kStage, fo.row_frag[j]);
      __builtin_amdgcn_sched_barrier(0);
      dkacc[j % DB] = mfma(tq1[j / DB][j % DB], dsb1[j / DB], dkacc[j % DB]);
      da[j] = lds_read_frag(smem + (3 - ST) * kStage, fo.row_frag[j]);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  int heads_left = hpu, st = 0;
  if (n_steps == 1 && hpu == 1) tickets.step(0);
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
  auto body = [&](auto stage_c) __attribute__((always_inline)) {
    const int q0 = to_next();
    if (q0 < wave_kv0 + 32 || q0 + kStep > it.doc_end) stage(q0, stage_c, std::true_type{});
    else stage(q0, stage_c, std::false_type{});
  };
  auto idle = [&]() __attribute__((always_inline)) {   // a stage without keys that its queries may see: loads and barrier only
    to_next();
    if (st & 1) all_pieces<1>(lds, wave);
    else all_pieces<0>(lds, wave);
    wait_vm<0>();
    __syncthreads();
  };
  // every query of a chain's first step lies before the keys of the upper two waves
  const int begin = it.step_begin == 0 && wave >= 2 ? 1 : 0;
  for (;;) {
    __syncthreads();
    if (begin) idle();
    if (wave_active && st < n_steps) {
      const char* const qt = smem + begin * kStage;
      if (begin) read_ahead_stats(std::integral_constant<int, 1>{}); else read_ahead_stats(std::integral_constant<int, 0>{});
      static_for<KK>([&](auto kk) __attribute__((always_inline)) {
        qa[kk] = lds_read_frag(qt, fo.row_frag[kk]);
        da[kk] = lds_read_frag(qt + NS * kStage, fo.row_frag[kk]);
      });
      int skip = begin;
      for (;;) {
        if (!skip) {
          body(std::integral_constant<int, 0>{});
          if (st >= n_steps) break;
        }
        skip = 0;
        body(std::integral_constant<int, 1>{});
        if (st >= n_steps) break;
      }
    }
    while (st < n_steps) idle();
    if (--heads_left == 0) break;
    __syncthreads();   // the last stage's read-ahead
    start(a, head + hpu - heads_left, wave);
    st = 0;
    if (n_steps == 1 && heads_left == 1) tickets.step(0);
    all_pieces<0>(lds, wave);
    wait_vm<0>();
  }
  }
};

template <int D>
__device__ __forceinline__ void store_dkv(const BwdArgs<D>& a, const varlen_attn_unit& it, int head, char* tile, const f32x16 (&dkacc)[D / 32],
                                          const f32x16 (&dvacc)[D / 32]) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (it.slot >= 0) {
    float* part = a.col_partials + ((size_t)it.slot * a.Hq + head) * 2 * frag_floats<D>();
    store_frag<D>(part, dkacc, wave, lane);
    store_frag<D>(part + frag_floats<D>(), dvacc, wave, lane);
  } else {
    const size_t first = ((size_t)(it.row0 + 32 * wave) * a.Hkv + head / (a.Hq / a.Hkv)) * D;
    const int rows = it.doc_end - it.row0 - 32 * wave;
    store_rows<D>(tile, a.dk + first, (size_t)a.Hkv * D, rows, dkacc, lane, a.scale);
    asm volatile("" ::: "memory");   // (one tile for both: the LDS serves a wave's accesses in order)
    store_rows<D>(tile, a.dv + first, (size_t)a.Hkv * D, rows, dvacc, lane, 1.0f);
  }
}

template <int D>
__global__ void __launch_bounds__(kThreads, 1) bwd_pool_kernel(BwdArgs<D> a) {
  __shared__ __attribute__((aligned(1024))) char smem[BwdLds<D>::kBytes];
  __shared__ __attribute__((aligned(1024))) char out_tiles[4 * RowTile<D>::kBytes];
  __shared__ int ticket;
  const int hpu = a.hdr->col_heads_per_unit, n_col = a.hdr->n_col_units;
  // a plan that was made for two kernels has no dQ units of its own: the row units
  const bool own_dq = a.hdr->n_dq_units > 0;
  const int n_dq = own_dq ? a.hdr->n_dq_units : a.hdr->n_row_units;
  const varlen_attn_unit* const dq_units = own_dq ? a.dq_units : a.row_units;
  if (n_col == 0) return;   // nothing planned
  TicketGroup g;
  g.init(blockIdx.x, gridDim.x, a.Hq, hpu, n_col, n_dq);
  if (g.first >= g.total) return;
  char* const tile = out_tiles + (threadIdx.x >> 6) * RowTile<D>::kBytes;
  FragOffsets<D> fo;
  fo.init(threadIdx.x & 63);
  Tickets tickets{a.tickets + g.index, &ticket, 0};
  // the units do not change while the kernel runs: scalar loads
  typedef const __attribute__((address_space(4))) varlen_attn_unit* constant_units;
  auto load_unit = [&](const varlen_attn_unit* units, int i) __attribute__((always_inline)) {
    const constant_units u = (constant_units)(size_t)units;
    return varlen_attn_unit{u[i].row0, u[i].doc_start, u[i].doc_end, u[i].step_begin, u[i].step_end, u[i].slot, 0, 0};
  };
  DqUnit<D> row;
  int t = g.first, unit, head;
  g.decode(t, unit, head);
  if (t < g.n_col) {
    DkvUnit<D> col;
    col.open(a, load_unit(a.col_units, unit), head, smem);
    f32x16 dkacc[D / 32], dvacc[D / 32];
#pragma unroll 1
    for (;;) {
      wait_all_vm_visible();
      col.sweep(a, hpu, smem, fo, dkacc, dvacc, tickets);
      const varlen_attn_unit done = col.it;
      const int done_head = col.head;
      t = g.members + tickets.take();
      g.decode(t, unit, head);
      if (t < g.n_col) col.open(a, load_unit(a.col_units, unit), head, smem);
      store_dkv<D>(a, done, done_head, tile, dkacc, dvacc);
      if (t >= g.n_col) break;
    }
    if (t >= g.total) return;
  }
  row.open(a, load_unit(dq_units, unit), head, smem);
  f32x16 acc[D / 32];
#pragma unroll 1
  for (;;) {
    wait_all_vm_visible();
    row.sweep(a, smem, fo, acc, tickets);
    const varlen_attn_unit done = row.it;
    const int done_head = row.head;
    t = g.members + tickets.take();
    if (t < g.total) {
      g.decode(t, unit, head);
      row.open(a, load_unit(dq_units, unit), head, smem);
    }
    store_dq<D>(a, done, done_head, tile, acc);
    if (t >= g.total) break;
  }
}

// Sums of the partial results of the pool, dealt as in fwd_combine_kernel: [dK | dV] of cut or grouped column tiles by the workgroups from the
// front, dQ of cut row tiles by the workgroups from the back.
template <int D>
__global__ void __launch_bounds__(kThreads)
bwd_pool_combine_kernel(const varlen_attn_plan_header* __restrict__ hdr, const varlen_attn_combine_item* __restrict__ col_items,
                        int max_col, const float* __restrict__ col_partials, const varlen_attn_combine_item* __restrict__ dq_items,
                        int max_row, const float* __restrict__ row_partials, __bf16* __restrict__ dq, __bf16* __restrict__ dk,
                        __bf16* __restrict__ dv, int Hq, int Hkv, float scale) {
  constexpr int DB = D / 32, kWavePieces = 4 * DB / 2;
  constexpr int kFlight = 4;
  using Tile = RowTile<64>;
  __shared__ __attribute__((aligned(16))) char tiles[2][Tile::kBytes];
  int buf = 0;
  const int lane = threadIdx.x & 63, rq = threadIdx.x >> 6, h = lane >> 5, c = lane & 31;
  const int n_col = min(hdr->n_col_combine, max_col), n_row = min(hdr->n_dq_combine, max_row), hpu = hdr->col_heads_per_unit;
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
