// Forward kernel and the reduction of its cut chains.
#ifndef VARLEN_ATTN_FWD_HPP_
#define VARLEN_ATTN_FWD_HPP_

#include "tiles.hpp"
#include "staging.hpp"
#include "fragments.hpp"
#include "plan.hpp"

namespace {

// ----------------------------------------------------------------------------------------
// Forward.  One workgroup per (row unit, q head); wave w owns query rows row0 + 32w .. +31.
// Computes S^T = K Q^T so that a query is a lane column; online softmax in the exp2 domain
// against a reference that is only renewed when it must be; O^T += V^T P^T.  A unit that covers its
// whole chain normalises and stores O and LSE; otherwise it stores the unnormalised accumulator
// with its reference and row sum for fwd_combine_kernel.
// ----------------------------------------------------------------------------------------
template <int D, bool SELF>
__global__ void __launch_bounds__(kThreads, 2)
fwd_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
           const varlen_attn_plan_header* __restrict__ hdr,
           const varlen_attn_unit* __restrict__ units, __bf16* __restrict__ o,
           float* __restrict__ lse, float* __restrict__ partials, int N, int Hq, int Hkv,
           float scale, int max_units, PlanArgs plan) {
  constexpr int KK = D / 16, DB = D / 32;
  constexpr int NS = 4;                              // pipeline stages of 32 keys
  constexpr int kStageBytes = kSub * D * 2;
  constexpr int LPS = 2 * StageLoader<D>::kPerWave;  // DMA loads per thread per stage (K and V)
  __shared__ __attribute__((aligned(1024))) char smem[2 * NS * kStageBytes];  // K stages, V stages

  int unit_idx, head;
  varlen_attn_unit it;
  if (SELF) {
    // Small microbatch: no plan launch in front.  Workgroup 0 makes the plan (for the reduction
    // of this forward and for the backward) while the others work out their own unit from
    // cu_seqlens by the plan's rules (the order: derive_row_unit).
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
    // (scalar registers again: everything derived from the unit stays wave-uniform)
    it = varlen_attn_unit{__builtin_amdgcn_readfirstlane(own_unit.row0), __builtin_amdgcn_readfirstlane(own_unit.doc_start),
                          __builtin_amdgcn_readfirstlane(own_unit.doc_end), __builtin_amdgcn_readfirstlane(own_unit.step_begin),
                          __builtin_amdgcn_readfirstlane(own_unit.step_end), __builtin_amdgcn_readfirstlane(own_unit.slot),
                          __builtin_amdgcn_readfirstlane(own_unit.cost), 0};
  } else {
    decode_block(blockIdx.x, Hq, unit_idx, head);
    // both loads in flight together; the unit array always has max_units >= grid / Hq entries
    const int n_units = hdr->n_row_units;
    it = units[min(unit_idx, max_units - 1)];
    if (unit_idx >= n_units) return;
  }
  const int kvh = head / (Hq / Hkv);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, c = lane & 31;
  const float cs = scale * kLog2e;

  const int wave_row0 = it.row0 + 32 * wave;
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
  const unsigned lds_k = lds_addr_of(smem), lds_v = lds_k + NS * kStageBytes;

  StageLoader<D> loader;
  loader.init(wave, lane, (unsigned)(kv_stride * 2));
  // stages are issued in order, one call per sub-step: the wave-uniform addresses of the next
  // stage's first K and V rows live in scalar registers and move on by one stage per call
  const unsigned long long kStageStride = (unsigned long long)kSub * (kv_stride * 2);
  unsigned long long k_next = uniform64(reinterpret_cast<const char*>(kbase) + (size_t)kv_begin * (kv_stride * 2));
  unsigned long long v_next = uniform64(reinterpret_cast<const char*>(vbase) + (size_t)kv_begin * (kv_stride * 2));
  auto issue = [&](int sub, int stage) {
    const int row0 = kv_begin + kSub * min(sub, n_sub - 1);
    loader.issue_at(k_next, row0, it.doc_end - 1, lds_k + stage * kStageBytes, wave);
    loader.issue_at(v_next, row0, it.doc_end - 1, lds_v + stage * kStageBytes, wave);
    if (sub < n_sub - 1) { k_next += kStageStride; v_next += kStageStride; }
  };
#pragma unroll
  for (int st = 0; st < NS - 1; ++st) issue(st, st);

  bf16x8 qf[KK];
  load_row_frags<D>(q + ((size_t)min(my_row, it.doc_end - 1) * Hq + head) * D, h, qf);
  FragOffsets<D> fo;
  fo.init(lane);
  // Let the compiler see its own loads complete here, once; otherwise it keeps a vmcnt(0)
  // for them inside the loop, which would also wait for every prefetch in flight.
  wait_all_vm_visible();
  pin_frags(qf);

  f32x16 oacc[DB];
#pragma unroll
  for (int i = 0; i < DB; ++i) oacc[i] = f32x16(0.f);
  float m_run = -INFINITY, l_run = 0.f;

  // Reference m of the exponentials: any m with 2^(s - m) far from overflow gives the same O and LSE
  // up to rounding.  It is the row's maximum over the first sub-step (so that a row of one key has
  // P = 1), and stays until the row sum of a sub-step, which is needed anyway, exceeds 2^8: only
  // then are the scores formed again, their maximum taken and O and the row sum rescaled.  Against
  // a maximum in every sub-step that leaves out 15 of 85 vector instructions and a chain of 17
  // dependent ones between the two contractions: 422 -> 410 us at 32768 tokens in 11 documents
  // (205e6 pairs, 4 heads of 128), 31.1 -> 30.3 us at 8192 tokens (7.1e6 pairs).
  auto scores = [&](const char* kt) __attribute__((always_inline)) {
    f32x16 s = f32x16(0.f);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) s = mfma(lds_read_frag(kt, fo.row_frag[kk]), qf[kk], s);
    return s;
  };
  auto mask = [&](f32x16& s, int kv0) __attribute__((always_inline)) {
    if (kv0 + kSub - 1 > wave_row0) {  // touches the diagonal for some row
      const int t = my_row - kv0 - 4 * h;  // key offset 8 (r / 4) + r % 4 is allowed iff <= t
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r / 4) + (r % 4) > t) s[r] = -INFINITY;
    }
  };
  auto row_max = [&](const f32x16& s) __attribute__((always_inline)) {
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = __builtin_fmaxf(mx, s[r]);
    return half_max(mx) * cs;
  };
  // s -> 2^(s cs - m), returns the sum over this lane's keys
  auto exponentials = [&](f32x16& s) __attribute__((always_inline)) {
    float ps[4];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], cs, -m_run));
      ps[r & 3] = r < 4 ? s[r] : ps[r & 3] + s[r];
    }
    return (ps[0] + ps[1]) + (ps[2] + ps[3]);
  };
  // one sub-step: 32 keys against this wave's 32 queries, stage index known at compile time
  auto compute = [&](int sub, auto stage_c) {
    constexpr int ST = decltype(stage_c)::value;
    const int kv0 = kv_begin + kSub * sub;
    if (!(wave_active && kv0 <= wave_last_row)) return;
    const char* kt = smem + ST * kStageBytes;
    const char* vt = smem + (NS + ST) * kStageBytes;
    __builtin_amdgcn_s_setprio(2);   // matrix phases win the issue slot over the other wave's softmax
    f32x16 s = scores(kt);
    __builtin_amdgcn_s_setprio(0);
    // the transposed V fragments of the second contraction are requested before the softmax
    // arithmetic, so that they arrive behind it
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 vtf[2][DB];
#pragma unroll
    for (int cc = 0; cc < 2; ++cc)
#pragma unroll
      for (int db = 0; db < DB; ++db) vtf[cc][db] = read_trans<D>(vt, fo, cc, db);
    __builtin_amdgcn_sched_barrier(0);
    mask(s, kv0);
    if (ST == 0 && sub == 0) m_run = row_max(s);
    float psum = exponentials(s);
    if (__any(!(psum <= kRefSumMax))) {   // rare (NaN among the scores comes here as well)
      s = scores(kt);
      mask(s, kv0);
      const float m_new = __builtin_fmaxf(m_run, row_max(s) + kRefRoom);
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[i][r] *= alpha;
      psum = exponentials(s);
    }
    l_run += psum;
    __builtin_amdgcn_s_setprio(2);
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
      const bf16x8 pb = pack8(s, 8 * cc);
#pragma unroll
      for (int db = 0; db < DB; ++db) oacc[db] = mfma(vtf[cc][db], pb, oacc[db]);
    }
    __builtin_amdgcn_s_setprio(0);
  };
  // iteration `sub`: its stage has landed once at most NS-2 newer stages are in flight; the
  // barrier also tells that every wave is done with the stage about to be refilled
  auto body = [&](int sub, auto stage_c) {
    constexpr int ST = decltype(stage_c)::value;
    wait_vm<(NS - 2) * LPS>();
    __syncthreads();
    issue(sub + NS - 1, (ST + NS - 1) % NS);
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
    // a wave that saw no key in this chunk leaves the neutral element (0, -inf, 0)
    float* part = partials + ((size_t)it.slot * Hq + head) * fwd_partial_floats<D>();
    store_frag<D>(part, oacc, wave, lane);
    part[frag_floats<D>() + tid] = m_run;
    part[frag_floats<D>() + kThreads + tid] = l_run;
    return;
  }
  __syncthreads();   // every wave is done with the stages
  if (!wave_active) return;
  const float l_tot = half_sum(l_run);
  store_rows<D>(smem + wave * RowTile<D>::kBytes, o + ((size_t)wave_row0 * Hq + head) * D, (size_t)Hq * D,
                it.doc_end - wave_row0, oacc, lane, 1.0f / l_tot);
  if (row_valid && h == 0) lse[(size_t)head * N + my_row] = (m_run + __builtin_amdgcn_logf(l_tot)) * kLn2;
}

// Sums the chunks of a cut row chain:  O = sum_c 2^(m_c - m) O_c / sum_c 2^(m_c - m) l_c.
// Elementwise over the fragment layout: a workgroup takes two neighbouring column blocks of one
// wave's rows of an (item, head), thread t of it float4 number t of both (so all loads are
// contiguous), chunks in chain order.  What bounds it is the chain of dependent round trips to
// data that another kernel has just written, so the loads of up to four chunks are in flight
// together, and a fixed number of workgroups walks over the items: launching one workgroup for
// every piece of every tile that might be cut took 5 us of the kernel's 7.  The 32 x 64 block of O
// is put together in LDS and stored in runs of 128 bytes.
template <int D>
__global__ void __launch_bounds__(kThreads)
fwd_combine_kernel(const varlen_attn_plan_header* __restrict__ hdr,
                   const varlen_attn_combine_item* __restrict__ items, int max_items,
                   const float* __restrict__ partials, __bf16* __restrict__ o,
                   float* __restrict__ lse, int N, int Hq) {
  constexpr int DB = D / 32;
  constexpr int kPieces = 4 * DB / 2;   // of an (item, head): 4 waves, pairs of column blocks
  constexpr int kFlight = 4;
  using Tile = RowTile<64>;
  __shared__ __attribute__((aligned(16))) char tiles[2][Tile::kBytes];
  int buf = 0;   // two tiles in turn: one barrier per item
  const int lane = threadIdx.x & 63, rq = threadIdx.x >> 6, h = lane >> 5, c = lane & 31;
  const size_t pstride = (size_t)Hq * fwd_partial_floats<D>();
  const int n_items = hdr->n_row_combine;
  for (int work = blockIdx.x; work < max_items * Hq * kPieces; work += gridDim.x) {
    const int piece = work % kPieces, rest = work / kPieces;
    const int idx = rest / Hq, head = rest % Hq;
    const varlen_attn_combine_item it = items[idx];   // in flight together with n_items
    if (idx >= n_items) return;
    const int wave = piece / (DB / 2), db = 2 * (piece % (DB / 2));
    const int row0 = it.row0 + 32 * wave, my_row = row0 + c;
    if (row0 >= it.doc_end) continue;   // (rows past the end inside the block: computed, not stored)
    const float* p0 = partials + ((size_t)it.slot0 * Hq + head) * fwd_partial_floats<D>();
    const float* st = p0 + frag_floats<D>() + wave * 64;  // m[lane], then l[lane] 256 floats on
    const float* x0 = p0 + (size_t)(wave * DB + db) * kThreads * 4 + (size_t)threadIdx.x * 4;
    float m = -INFINITY, l = 0.f;
    f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
#pragma unroll 1
    for (int ch = 0; ch < it.n_chunks; ch += kFlight) {
      float mc[kFlight], la[kFlight], lb[kFlight];
      f32x4 xa[kFlight], xb[kFlight];
      float m_new = m;
#pragma unroll
      for (int j = 0; j < kFlight; ++j) {
        mc[j] = -INFINITY; la[j] = lb[j] = 0.f; xa[j] = xb[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (ch + j < it.n_chunks) {   // the same for the whole workgroup
          const size_t off = (size_t)(ch + j) * pstride;
          mc[j] = st[off + lane];
          la[j] = st[off + kThreads + c];
          lb[j] = st[off + kThreads + 32 + c];
          xa[j] = *reinterpret_cast<const f32x4*>(x0 + off);
          xb[j] = *reinterpret_cast<const f32x4*>(x0 + off + kThreads * 4);
        }
      }
#pragma unroll
      for (int j = 0; j < kFlight; ++j) m_new = __builtin_fmaxf(m_new, mc[j]);
      if (ch > 0) {
        const float w = __builtin_amdgcn_exp2f(m - m_new);
        l *= w; acc0 *= w; acc1 *= w;
      }
      m = m_new;
#pragma unroll
      for (int j = 0; j < kFlight; ++j) {
        const float w = __builtin_amdgcn_exp2f(mc[j] - m);
        l += w * (la[j] + lb[j]);
        acc0 += w * xa[j];
        acc1 += w * xb[j];
      }
    }
    const float inv = 1.0f / l;
    Tile::put(tiles[buf], c, h, rq, pack4(acc0[0] * inv, acc0[1] * inv, acc0[2] * inv, acc0[3] * inv));
    Tile::put(tiles[buf], c, h, 4 + rq, pack4(acc1[0] * inv, acc1[1] * inv, acc1[2] * inv, acc1[3] * inv));
    __syncthreads();
    const int out_row = row0 + (threadIdx.x >> 3), chunk = threadIdx.x & 7;
    const uint4 w = Tile::get(tiles[buf], threadIdx.x >> 3, chunk);
    if (out_row < it.doc_end) *reinterpret_cast<uint4*>(o + ((size_t)out_row * Hq + head) * D + 32 * db + 8 * chunk) = w;
    buf ^= 1;
    if (db == 0 && rq == 0 && h == 0 && my_row < it.doc_end)
      lse[(size_t)head * N + my_row] = (m + __builtin_amdgcn_logf(l)) * kLn2;
  }
}

}  // namespace

#endif  // VARLEN_ATTN_FWD_HPP_
