// Forward with heads of 128: two waves of 64 rows.
#ifndef VARLEN_ATTN_FWD_WIDE_HPP_
#define VARLEN_ATTN_FWD_WIDE_HPP_

#include "tiles.hpp"
#include "staging.hpp"
#include "panels.hpp"
#include "fragments.hpp"
#include "plan.hpp"

namespace {

// ----------------------------------------------------------------------------------------
// The forward of fwd.hpp (same units, order, reference, partial results) with two waves a workgroup, one a SIMD: wave w owns
// rows row0 + 64 w .. + 63 as two blocks of 32, so that a fragment of K or V from LDS feeds two matrix instructions, and the
// substeps of 32 keys are pipelined by hand:
//   S of the next substep (16 matrix instructions) beside the upper 8 registers' exponentials of this one | check |
//   O += P V of this one (16) beside the lower 8 registers' exponentials of the next one; in the middle of it the wait and the barrier.
// One exponential (multiply-add, exp, sum, half a rounding: 30 of the 32 clocks that a matrix instruction takes) to a matrix
// instruction, held there by inline assembly: two beside one and none beside the next, which is what the compiler makes of the
// same source, took 1.07 times as long (424 -> 398 us on the first of the packs below).  K and V are double-buffered in steps of
// 64 keys (32 KB each); what a barrier frees is requested behind it and waited for two barriers on.  What bounds it: vector work
// and matrix work that are equally long, and on large microbatches the clock.  Forward alone, two-wave SIMDs / here: 32768
// tokens in 11 documents (4 heads) 435 -> 398 us, 32768 in 35 117 -> 110, 16384 (8 q heads on one) 169 -> 160; whole steps 1557
// -> 1524, 402 -> 392, 595 -> 582, 131072 in one document 30.7 -> 29.9 ms.  First loads and last stores have no other wave to
// hide behind, which short chains pay for: wide_forward() in varlen_attn.hip.
// ----------------------------------------------------------------------------------------
template <bool SELF>
__global__ void __launch_bounds__(128, 1)
fwd_wide_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
                const varlen_attn_plan_header* __restrict__ hdr, const varlen_attn_unit* __restrict__ units, __bf16* __restrict__ o,
                float* __restrict__ lse, float* __restrict__ partials, int N, int Hq, int Hkv, float scale, int max_units, PlanArgs plan) {
  constexpr int D = 128, KK = D / 16, DB = D / 32, kTileBytes = kStep * D * 2, kStage = 2 * kTileBytes, kPanel = PanelOffsets<D>::kPanel;
  __shared__ __attribute__((aligned(1024))) char smem[2 * kStage];

  int unit_idx, head;
  varlen_attn_unit it;
  if (SELF) {
    __shared__ varlen_attn_unit own_unit;
    __shared__ int own_valid;
    if (blockIdx.x == 0) {
      if (threadIdx.x < kPlanThreadsSmall) plan_body<kPlanThreadsSmall>(plan);
      return;
    }
    decode_block(blockIdx.x - 1, Hq, unit_idx, head);
    if (threadIdx.x < 64) {
      varlen_attn_unit mine;
      const bool ok = derive_row_unit(plan.cu, plan.B, plan.N, Hq, plan.no_split, plan.rule[0], plan.force_ch[0],
                                      plan.slots_cap, unit_idx, plan.longest_first, threadIdx.x, mine);
      if (threadIdx.x == 0) { own_valid = ok ? 1 : 0; if (ok) own_unit = mine; }
    }
    __syncthreads();
    if (!own_valid) return;
    it = varlen_attn_unit{__builtin_amdgcn_readfirstlane(own_unit.row0), __builtin_amdgcn_readfirstlane(own_unit.doc_start),
                          __builtin_amdgcn_readfirstlane(own_unit.doc_end), __builtin_amdgcn_readfirstlane(own_unit.step_begin),
                          __builtin_amdgcn_readfirstlane(own_unit.step_end), __builtin_amdgcn_readfirstlane(own_unit.slot),
                          __builtin_amdgcn_readfirstlane(own_unit.cost), 0};
  } else {
    decode_block(blockIdx.x, Hq, unit_idx, head);
    const int n_units = hdr->n_row_units;
    it = units[min(unit_idx, max_units - 1)];
    if (unit_idx >= n_units) return;
  }
  const int kvh = head / (Hq / Hkv);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), h = lane >> 5, c = lane & 31;
  const float cs = scale * kLog2e;
  const int wave_row0 = it.row0 + 64 * wave;
  const bool wave_active = wave_row0 < it.doc_end;
  const int kv_begin = it.doc_start + it.step_begin * kStep;
  const int wg_last_row = min(it.row0 + kTile, it.doc_end) - 1;
  const int kv_end = min(it.doc_start + it.step_end * kStep, wg_last_row + 1);
  const int n_steps = (kv_end - kv_begin + kStep - 1) / kStep;
  // steps in front of this wave's rows, all keys of which they see; then, unless the chunk ends before, the step on the diagonal
  const int full = wave_active ? min(n_steps, max(0, (wave_row0 - kv_begin) / kStep)) : 0;
  const bool diagonal = wave_active && wave_row0 >= kv_begin && full < n_steps;

  const unsigned stride = (unsigned)(Hkv * D * 2);
  const unsigned long long stage_stride = (unsigned long long)kStep * stride;
  unsigned long long k_next = uniform64(k + ((size_t)kv_begin * Hkv + kvh) * D);
  unsigned long long v_next = uniform64(v + ((size_t)kv_begin * Hkv + kvh) * D);
  const unsigned col = (unsigned)(((lane ^ (lane >> 4)) & 3) * 16);
  const unsigned own = (unsigned)(16 * wave + (lane >> 2)) * stride + col;
  const unsigned lds = lds_addr_of(smem) + wave * 1024;
  // rows of a stage above the document's last are clamped to it
  auto last_of = [&](int step) { return (unsigned)min(it.doc_end - 1 - (kv_begin + kStep * step), kStep - 1) * stride + col; };
  // piece P of a tile's eight: panel P / 2, rows 16 wave .. or 32 further on
  auto aim_piece = [&](auto p_c, unsigned to) __attribute__((always_inline)) {
    constexpr int P = decltype(p_c)::value;
    asm volatile("s_add_u32 m0, %0, %1" : : "s"(to), "n"((P >> 1) * (kPanel - 64) + (P & 1) * 2048) : "scc");
  };
  auto load_piece = [&](auto p_c, unsigned long long base, unsigned off0, unsigned off1) __attribute__((always_inline)) {
    constexpr int P = decltype(p_c)::value;
    asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" : : "v"(P & 1 ? off1 : off0), "s"(base), "n"(64 * (P >> 1)) : "memory");
  };
  auto load_tile = [&](unsigned long long base, unsigned last, unsigned to) __attribute__((always_inline)) {
    const unsigned off0 = min(own, last), off1 = min(own + 32 * stride, last);
    static_for<8>([&](auto p) __attribute__((always_inline)) {
      aim_piece(p, to);
      asm volatile("s_nop 0");
      load_piece(p, base, off0, off1);
    });
  };
  int k_step = 0, v_step = 0;   // whose tiles k_next, v_next are
  auto next_k = [&]() { if (k_step < n_steps - 1) { ++k_step; k_next += stage_stride; } };
  auto next_v = [&]() { if (v_step < n_steps - 1) { ++v_step; v_next += stage_stride; } };
  load_tile(k_next, last_of(0), lds);
  load_tile(v_next, last_of(0), lds + kTileBytes);
  next_k();
  next_v();
  bf16x8 qf[2][KK];
#pragma unroll
  for (int b = 0; b < 2; ++b) load_row_frags<D>(q + ((size_t)min(wave_row0 + 32 * b + c, it.doc_end - 1) * Hq + head) * D, h, qf[b]);
  f32x16 acc[2][DB];
  {
    const bf16x8 zeros = zero_frag();
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < DB; ++i) acc_zero(acc[b][i], zeros);
  }
  wait_all_vm_visible();
  pin_frags_acc(qf[0]);
  pin_frags_acc(qf[1]);
  load_tile(k_next, last_of(k_step), lds + kStage);
  next_k();
  __syncthreads();

  PanelOffsets<D> fo;
  fo.init(lane, 0);
  constexpr int kHalfOff = 32 * 64;
  const int tri = c - 4 * h;   // of a block on the diagonal, allowed: 8 (r / 4) + r % 4 <= tri
  float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.f, 0.f}, psum[2] = {0.f, 0.f};
  bf16x8 ka[KK / 2], pb0[2], pb1[2], pb0n[2];
  f32x16 sa[2], sb[2];
  auto fence = []() __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };
  auto mask = [&](f32x16& s) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (8 * (r >> 2) + (r & 3) > tri) s[r] = -INFINITY;
  };
  auto row_max = [&](const f32x16& s) __attribute__((always_inline)) {
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = __builtin_fmaxf(mx, s[r]);
    return half_max(mx) * cs;
  };
  // 2^(s cs - m) of register r, held in its place among the matrix instructions (a fence alone does not hold arithmetic); its sum and
  // rounded pair follow behind the next one's, so that nobody waits for it
  auto exponential = [&](f32x16& s, int b, int r) __attribute__((always_inline)) {
    float x = s[r];
    asm volatile("v_fma_f32 %0, %0, %1, -%2\n\tv_exp_f32 %0, %0" : "+v"(x) : "s"(cs), "v"(m[b]));
    s[r] = x;
  };
  auto add_up = [&](const f32x16& s, int b, int r, bf16x8& out) __attribute__((always_inline)) {
    const float e = s[r];
    psum[b] = r == 0 ? e : psum[b] + e;
    if (r & 1) {
      const f32x2 p = {s[r - 1], e};
      const bf16x2 p2 = __builtin_convertvector(p, bf16x2);
      out[(r & 7) - 1] = p2[0];
      out[r & 7] = p2[1];
    }
  };
  // item i of the 16 of one half of the registers, blocks FIRST .. 1
  auto half_items = [&](auto i_c, auto first_c, auto upper_c, f32x16 (&s)[2], bf16x8 (&out)[2]) __attribute__((always_inline)) {
    constexpr int i = decltype(i_c)::value, first = decltype(first_c)::value, base = decltype(upper_c)::value ? 8 : 0, p = i - 1;
    if constexpr (i < 16 && (i >> 3) >= first) exponential(s[i >> 3], i >> 3, base + (i & 7));
    if constexpr (p >= 0 && (p >> 3) >= first) add_up(s[p >> 3], p >> 3, base + (p & 7), out[p >> 3]);
  };
  // O, the row sum and this substep's as of a new reference
  auto rescale = [&](int b, float m_new) __attribute__((always_inline)) {
    const float alpha = __builtin_amdgcn_exp2f(m[b] - m_new);
    m[b] = m_new;
    l[b] *= alpha;
    psum[b] *= alpha;
#pragma unroll
    for (int i = 0; i < DB; ++i) {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[b][i][r] *= alpha;
      asm volatile("" : "+a"(acc[b][i]));
      fence();
    }
  };
  // Rare: block b against a new reference.  Its scores are gone by now and the probabilities at hand are scaled, which gives a
  // row's largest the same 2^-12 exactly.  To form the scores again from memory (the K tile may be landing on already) stops
  // both waves for the time of a load, and is done for sums beyond 2^100, whose scaling would leave the range, and NaN.
  // Forward at 32768 tokens in 35 documents, 16384 (8 q heads on one) and 32768 in 11, scores with a standard deviation of 9,
  // from memory each time 153.6, 191.6 and 472 us, scaled 126.0, 166.3 and 437; with a standard deviation of 1 114.1, 148.9 and
  // 402, scaled 113.3, 148.8 and 402.
  auto renew = [&](f32x16& s, int b, int kv0, bool triangle) __attribute__((always_inline)) {
    if (__builtin_expect(__any(!(psum[b] <= 0x1p100f)), 0)) {
      const __bf16* row = k + ((size_t)min(kv0 + c, it.doc_end - 1) * Hkv + kvh) * D + 8 * h;
      f32x16 x = f32x16(0.f);
      static_for<KK>([&](auto i_c) __attribute__((always_inline)) {
        constexpr int i = decltype(i_c)::value;
        x = mfma(__builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(row + 16 * i)), qf[b][i], x);
        fence();
      });
      if (triangle) mask(x);
      rescale(b, __builtin_fmaxf(m[b], row_max(x) + kRefRoom));
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        exponential(x, b, r);
        add_up(x, b, r, r < 8 ? pb0[b] : pb1[b]);
      }
      return;
    }
    float top = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) top = __builtin_fmaxf(top, s[r]);
    const float m_old = m[b], m_new = __builtin_fmaxf(m_old, m_old + (__builtin_amdgcn_logf(half_max(top)) + kRefRoom));
    const float alpha = __builtin_amdgcn_exp2f(m_old - m_new);
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] *= alpha;
    pb0[b] = pack8(s, 0);
    pb1[b] = pack8(s, 8);
    rescale(b, m_new);
  };
  int t = 0;
  // Substep x = 32 HALF .. of step t: S of the next substep beside the upper half of x's exponentials, then O += P V of x
  // beside the lower half of the next one's.
  auto iter = [&](auto half_c, auto diag_c, f32x16 (&cur)[2], f32x16 (&nxt)[2], bool next_diag) __attribute__((always_inline)) {
    constexpr int HALF = decltype(half_c)::value;
    constexpr bool DIAG = decltype(diag_c)::value, NEXT = !(DIAG && HALF);
    constexpr int NB = DIAG && !HALF ? 1 : 0, CB = DIAG && HALF ? 1 : 0;   // first block that the next substep, that this one is for
    const char* const kt = smem + (HALF ? 0 : kHalfOff);
    const char* const vt = smem + kTileBytes + (HALF ? kHalfOff : 0);
    const unsigned to = lds + (HALF ? (t & 1) * kStage : ((t + 1) & 1) * kStage + kTileBytes);
    const unsigned long long base = HALF ? k_next : v_next;
    const unsigned last = last_of(HALF ? k_step : v_step), off0 = min(own, last), off1 = min(own + 32 * stride, last);
    bf16x8 kf[KK], vf[2][DB];
    auto next_v_frag = [&](auto j_c) __attribute__((always_inline)) {
      constexpr int j = decltype(j_c)::value;
      if constexpr (j >= 0 && j < 2 * DB) vf[j / DB][j % DB] = fo.trans_frag(vt, j / DB, j % DB);
    };
    auto upper = [&](auto i_c) __attribute__((always_inline)) {   // item i of 16
      half_items(i_c, std::integral_constant<int, CB>{}, std::true_type{}, cur, pb1);
    };
#pragma unroll
    for (int i = 0; i < KK / 2; ++i) kf[i] = ka[i];
    static_for<KK>([&](auto kk_c) __attribute__((always_inline)) {
      constexpr int kk = decltype(kk_c)::value;
      aim_piece(kk_c, to);
      if constexpr (NEXT && NB == 0) {
        if constexpr (kk == 0) mfma_vgpr_agpr_first(nxt[0], kf[kk], qf[0][kk]);
        else mfma_vgpr_agpr(nxt[0], kf[kk], qf[0][kk]);
      } else {
        // (a load to LDS takes m0 one wait state behind its write at the earliest; elsewhere the matrix instruction is that)
        asm volatile("s_nop 0");
      }
      if constexpr (NEXT && kk < KK / 2) kf[kk + KK / 2] = fo.row_frag(kt, kk + KK / 2);
      upper(std::integral_constant<int, 2 * kk>{});
      fence();
      load_piece(kk_c, base, off0, off1);
      if constexpr (NEXT) {
        if constexpr (kk == 0) mfma_vgpr_agpr_first(nxt[1], kf[kk], qf[1][kk]);
        else mfma_vgpr_agpr(nxt[1], kf[kk], qf[1][kk]);
      }
      next_v_frag(std::integral_constant<int, kk - 4>{});
      upper(std::integral_constant<int, 2 * kk + 1>{});
      fence();
    });
    upper(std::integral_constant<int, 16>{});
    if (HALF) next_k(); else next_v();
    {
      bool bad = !(psum[1] <= kRefSumMax);
      if (CB == 0) bad = bad || !(psum[0] <= kRefSumMax);
      if (__builtin_expect(__any(bad), 0)) {
        const int kv0 = kv_begin + kStep * t + 32 * HALF;
        if (CB == 0)
          if (__any(!(psum[0] <= kRefSumMax))) renew(cur[0], 0, kv0, DIAG);
        if (__any(!(psum[1] <= kRefSumMax))) renew(cur[1], 1, kv0, DIAG && HALF);
      }
    }
    if (CB == 0) l[0] += psum[0];
    l[1] += psum[1];
    static_for<2 * DB>([&](auto j_c) __attribute__((always_inline)) {
      constexpr int j = decltype(j_c)::value, cc = j / DB, db = j % DB;
      if constexpr (j == 5) {
        wait_vm<8>();
        __syncthreads();
        if constexpr (!HALF) { fo.row[0] ^= kStage; fo.row[1] ^= kStage; }
      }
      if constexpr (CB == 0) acc[0][db] = mfma(vf[cc][db], cc ? pb1[0] : pb0[0], acc[0][db]);
      next_v_frag(std::integral_constant<int, j + 4>{});
      if constexpr (j >= 5 && !(DIAG && !HALF)) {
        const char* const kn = smem + (HALF ? kHalfOff : 0);
        if constexpr (j == 5) { ka[0] = fo.row_frag(kn, 0); ka[1] = fo.row_frag(kn, 1); }
        else ka[j - 4] = fo.row_frag(kn, j - 4);
      }
      auto lower = [&](auto i_c) __attribute__((always_inline)) {
        if constexpr (NEXT) half_items(i_c, std::integral_constant<int, NB>{}, std::false_type{}, nxt, pb0n);
      };
      if constexpr (j == 1 && NEXT) {
        if constexpr (DIAG && !HALF) mask(nxt[1]);
        else if constexpr (HALF) {
          if (next_diag) {
            asm volatile("");   // a branch
            mask(nxt[0]);
          }
        }
      }
      if constexpr (j >= 1) lower(std::integral_constant<int, 2 * j - 2>{});
      if constexpr (j == 7) lower(std::integral_constant<int, 13>{});
      fence();
      acc[1][db] = mfma(vf[cc][db], cc ? pb1[1] : pb0[1], acc[1][db]);
      if constexpr (j >= 1 && j < 7) lower(std::integral_constant<int, 2 * j - 1>{});
      if constexpr (j == 7) static_for<3>([&](auto x) __attribute__((always_inline)) { lower(std::integral_constant<int, 14 + decltype(x)::value>{}); });
      fence();
    });
    if constexpr (HALF) { fo.trans[0] ^= kStage; fo.trans[1] ^= kStage; ++t; }
    if constexpr (NEXT) { pb0[0] = pb0n[0]; pb0[1] = pb0n[1]; }
  };
  if (full > 0 || diagonal) {
    {
      bf16x8 kf[KK];
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) kf[kk] = fo.row_frag(smem, kk);
#pragma unroll
      for (int kk = 0; kk < KK / 2; ++kk) ka[kk] = fo.row_frag(smem + kHalfOff, kk);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        mfma_vgpr_agpr_first(sa[b], kf[0], qf[b][0]);
#pragma unroll
        for (int kk = 1; kk < KK; ++kk) mfma_vgpr_agpr(sa[b], kf[kk], qf[b][kk]);
      }
      mfma_vgpr_settle();
      asm volatile("" : "+v"(sa[0]), "+v"(sa[1]));
      if (full == 0) mask(sa[0]);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        m[b] = row_max(sa[b]);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          exponential(sa[b], b, r);
          add_up(sa[b], b, r, pb0[b]);
        }
      }
      fence();
    }
#pragma unroll 1
    while (t < full) {
      iter(std::integral_constant<int, 0>{}, std::false_type{}, sa, sb, false);
      iter(std::integral_constant<int, 1>{}, std::false_type{}, sb, sa, t == full - 1);
    }
    if (diagonal) {
      iter(std::integral_constant<int, 0>{}, std::true_type{}, sa, sb, false);
      iter(std::integral_constant<int, 1>{}, std::true_type{}, sb, sa, false);
    }
  }
#pragma unroll 1
  while (t < n_steps) {   // steps without a key for this wave: loads and barriers only
    load_tile(v_next, last_of(v_step), lds + ((t + 1) & 1) * kStage + kTileBytes);
    next_v();
    wait_vm<8>();
    __syncthreads();
    load_tile(k_next, last_of(k_step), lds + (t & 1) * kStage);
    next_k();
    wait_vm<8>();
    __syncthreads();
    ++t;
  }
  wait_vm<0>();

  if (it.slot >= 0) {
    float* part = partials + ((size_t)it.slot * Hq + head) * fwd_partial_floats<D>();
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      store_frag<D>(part, acc[b], 2 * wave + b, lane);
      part[frag_floats<D>() + (2 * wave + b) * 64 + lane] = m[b];
      part[frag_floats<D>() + kThreads + (2 * wave + b) * 64 + lane] = l[b];
    }
    return;
  }
  __syncthreads();   // every wave is done with the stages
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int row0 = wave_row0 + 32 * b;
    if (row0 >= it.doc_end) break;
    const float l_tot = half_sum(l[b]);
    store_rows<D>(smem + (2 * wave + b) * RowTile<D>::kBytes, o + ((size_t)row0 * Hq + head) * D, (size_t)Hq * D, it.doc_end - row0, acc[b], lane,
                  1.0f / l_tot);
    if (row0 + c < it.doc_end && h == 0) lse[(size_t)head * N + row0 + c] = (m[b] + __builtin_amdgcn_logf(l_tot)) * kLn2;
  }
}

}  // namespace

#endif  // VARLEN_ATTN_FWD_WIDE_HPP_
