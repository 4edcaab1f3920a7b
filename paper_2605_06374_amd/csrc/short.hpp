// Forward and backward of small microbatches in one launch each.
#ifndef VARLEN_ATTN_SHORT_HPP_
#define VARLEN_ATTN_SHORT_HPP_

#include "tiles.hpp"
#include "staging.hpp"
#include "plan.hpp"

namespace {

// ----------------------------------------------------------------------------------------
// A microbatch of a few thousand tokens is bound by latency: launches, and the longest chain of
// a tile.  Here a workgroup owns 32 rows and its four waves share the chain of 32 x 32 blocks of
// those rows (wave w takes blocks w, w + 4, ...), so that a chain takes a quarter of its length;
// the four partial results meet in LDS.  No chain is cut across workgroups: no partial results in
// memory and no reduction launch, except for the q heads of a group in the backward, which store fp32
// [dK | dV] each and are added up by a second launch.  Every wave stages its blocks for itself, two in flight, without a
// barrier before the end.  D = rowsum(dO * O) is formed where it is used, so that dQ and dK / dV
// need no order between them and share one launch.
// The price is one read of K and V (Q, dO, O) per 32 rows instead of 128 and the LDS: one workgroup per CU
// at d = 128 (133 KB forward, 160 KB backward), two at d = 64.
// 777 tokens, 4 heads of 128, forward 14.5 -> 7.9 us (with the plan in workgroup 0 or its status word alone),
// backward 29.4 -> 10.5 us; 2048 tokens in 4 documents, 2 heads of 64, forward and backward 37.4 ->
// 27.9 us.  The rule by which a microbatch comes here is short_path() in varlen_attn.hip.
// ----------------------------------------------------------------------------------------
constexpr int kShortRows = 32;
constexpr float kShortLag = 8.f;   // the forward's running maximum may lag by 2^8 before O is rescaled

// The u-th 32-row tile of a microbatch of at most 64 documents, worked out by a whole wave from the
// documents that the plan kept or, while the plan is being made beside it (`planned` false), from
// cu_seqlens; every lane gets the answer.  False: malformed, nothing planned, or u past the last tile.
struct ShortTile { int row0, doc_start, doc_end; };
__device__ __forceinline__ bool derive_short_tile(const PlanArgs& plan, bool planned, int u, bool from_end,
                                                  int lane, ShortTile& out) {
  const int B = plan.B, N = plan.N;
  int s = 0, e = 0;
  if (planned) {
    if (lane < B) e = kept_ends(plan.hdr)[lane];
    s = __builtin_amdgcn_update_dpp(0, e, 0x138, 0xF, 0xF, true);   // wave_shr:1, 0 into lane 0
    if (lane >= B) s = 0;
  } else if (lane < B) { s = plan.cu[lane]; e = plan.cu[lane + 1]; }
  if (__any(lane < B && e < s) || lane_value(s, 0) != 0 || lane_value(e, B - 1) != N) return false;
  const int T = (e - s + kShortRows - 1) / kShortRows;
  const int incl = wave_inclusive_sum(T);
  const int total = lane_value(incl, 63);
  if (u >= total) return false;
  const int t = from_end ? total - 1 - u : u;
  const int doc = __popcll(__ballot(incl <= t));
  out.doc_start = lane_value(s, doc);
  out.doc_end = lane_value(e, doc);
  out.row0 = out.doc_start + (t - lane_value(incl - T, doc)) * kShortRows;
  return true;
}

// One wave's direct-to-LDS loads of a 32-row block of a [rows][D] tile.
template <int D>
struct BlockLoader {
  static constexpr int kRowsPerInstr = 1024 / (D * 2);            // 4 (D = 128), 8 (D = 64)
  static constexpr int kInstr = kShortRows / kRowsPerInstr;       // 8, 4
  static constexpr int kPeriod = kInstr / 2;                      // the swizzle repeats every 16 rows
  unsigned voff[kPeriod];
  unsigned stride_bytes;
  int lane;
  __device__ __forceinline__ void init(int lane_, unsigned stride_bytes_) {
    lane = lane_;
    stride_bytes = stride_bytes_;
#pragma unroll
    for (int j = 0; j < kPeriod; ++j) {
      const int r = kRowsPerInstr * j + lane / (D / 8);
      voff[j] = (unsigned)r * stride_bytes + (unsigned)(((lane % (D / 8)) ^ swz<D>(r)) * 16);
    }
  }
  // `first`: wave-uniform address of the block's first row; rows from `valid` on repeat the last one
  __device__ __forceinline__ void issue(unsigned long long first, int valid, unsigned lds) const {
    if (valid >= kShortRows) {
#pragma unroll
      for (int j = 0; j < kInstr; ++j)
        dma16(first + (unsigned long long)(j / kPeriod) * 16 * stride_bytes, voff[j % kPeriod], lds + j * 1024);
    } else {
#pragma unroll
      for (int j = 0; j < kInstr; ++j) {
        const int r = kRowsPerInstr * j + lane / (D / 8);
        const unsigned col = (unsigned)(((lane % (D / 8)) ^ swz<D>(r)) * 16);
        dma16(first, (unsigned)min(r, valid - 1) * stride_bytes + col, lds + j * 1024);
      }
    }
  }
};

// One wave's accumulator of a 32-row tile into its LDS region, in fragment order: float4 number
// (db * 4 + rq) * 64 + lane.
template <int D>
__device__ __forceinline__ void put_acc(char* region, const f32x16 (&acc)[D / 32], int lane, float mul) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) {
      const f32x4 t = {acc[db][4 * rq] * mul, acc[db][4 * rq + 1] * mul, acc[db][4 * rq + 2] * mul, acc[db][4 * rq + 3] * mul};
      *reinterpret_cast<f32x4*>(region + ((db * 4 + rq) * 64 + lane) * 16) = t;
    }
}
// Sum of the four waves' regions, float4 number `t`
template <int D>
__device__ __forceinline__ f32x4 sum_acc(const char* regions, int t) {
  f32x4 x = *reinterpret_cast<const f32x4*>(regions + t * 16);
#pragma unroll
  for (int w = 1; w < 4; ++w) x += *reinterpret_cast<const f32x4*>(regions + w * (kShortRows * D * 4) + t * 16);
  return x;
}

template <int D>
__global__ void __launch_bounds__(kThreads, D == 64 ? 2 : 1)
fwd_short_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
                 __bf16* __restrict__ o, float* __restrict__ lse, int Hq, int Hkv, float scale,
                 int plan_block, PlanArgs plan) {
  constexpr int KK = D / 16, DB = D / 32;
  constexpr int kBlockBytes = kShortRows * D * 2;
  constexpr int kWaveBytes = 4 * kBlockBytes;      // two stages of K and V
  __shared__ __attribute__((aligned(1024))) char smem[4 * kWaveBytes];
  __shared__ float stat_m[4][32], stat_l[4][32];

  if (plan_block && blockIdx.x == 0) {
    if (threadIdx.x < kPlanThreadsSmall) plan_body<kPlanThreadsSmall>(plan);
    return;
  }
  const int N = plan.N;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, c = lane & 31;
  int unit, head;
  decode_block(blockIdx.x - plan_block, Hq, unit, head);
  ShortTile it;
  if (!derive_short_tile(plan, !plan_block, unit, true, lane, it)) return;
  const int kvh = head / (Hq / Hkv);
  const int my_row = it.row0 + c;
  const bool row_valid = my_row < it.doc_end;
  const int n_blocks = (it.row0 - it.doc_start) / kShortRows + 1;   // the last one is the diagonal block
  const float cs = scale * kLog2e;

  BlockLoader<D> loader;
  const unsigned kv_stride = (unsigned)((size_t)Hkv * D * 2);
  loader.init(lane, kv_stride);
  const unsigned long long step = 4ull * kShortRows * kv_stride;
  unsigned long long k_next = uniform64(k + ((size_t)(it.doc_start + kShortRows * wave) * Hkv + kvh) * D);
  unsigned long long v_next = uniform64(v + ((size_t)(it.doc_start + kShortRows * wave) * Hkv + kvh) * D);
  char* const ring = smem + wave * kWaveBytes;
  const unsigned lds = lds_addr_of(smem) + wave * kWaveBytes;
  auto issue = [&](int block, int stage) __attribute__((always_inline)) {
    const int valid = it.doc_end - it.doc_start - kShortRows * block;
    loader.issue(k_next, valid, lds + stage * 2 * kBlockBytes);
    loader.issue(v_next, valid, lds + stage * 2 * kBlockBytes + kBlockBytes);
    k_next += step; v_next += step;
  };
  if (wave < n_blocks) issue(wave, 0);
  bf16x8 qf[KK];
  load_row_frags<D>(q + ((size_t)min(my_row, it.doc_end - 1) * Hq + head) * D, h, qf);
  FragOffsets<D> fo;
  fo.init(lane);
  wait_all_vm_visible();
  pin_frags(qf);

  f32x16 oacc[DB];
#pragma unroll
  for (int i = 0; i < DB; ++i) oacc[i] = f32x16(0.f);
  float m_run = -INFINITY, l_run = 0.f;
  int stage = 0;
#pragma unroll 1
  for (int j = wave; j < n_blocks; j += 4, stage ^= 1) {
    if (j + 4 < n_blocks) { issue(j + 4, stage ^ 1); wait_vm<2 * BlockLoader<D>::kInstr>(); }
    else wait_vm<0>();
    const char* kt = ring + stage * 2 * kBlockBytes;
    const char* vt = kt + kBlockBytes;
    f32x16 s;
    bf16x8 kf[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) kf[kk] = lds_read_frag(kt, fo.row_frag[kk]);
    __builtin_amdgcn_sched_barrier(0);
    static_for<KK>([&](auto kk) __attribute__((always_inline)) { mfma_vgpr_acc<kk == 0>(s, kf[kk], qf[kk]); });
    bf16x8 vtf[2][DB];
#pragma unroll
    for (int cc = 0; cc < 2; ++cc)
#pragma unroll
      for (int db = 0; db < DB; ++db) vtf[cc][db] = read_trans<D>(vt, fo, cc, db);
    mfma_vgpr_settle();
    if (j == n_blocks - 1) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r / 4) + (r % 4) > c - 4 * h) s[r] = -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = __builtin_fmaxf(mx, s[r]);
    const float m_new = __builtin_fmaxf(m_run, half_max(mx) * cs);
    if (__any(m_new > m_run + kShortLag)) {
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[i][r] *= alpha;
    }
    float ps[4];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], cs, -m_run));
      ps[r & 3] = r < 4 ? s[r] : ps[r & 3] + s[r];
    }
    l_run += (ps[0] + ps[1]) + (ps[2] + ps[3]);
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
      const bf16x8 pb = pack8(s, 8 * cc);
#pragma unroll
      for (int db = 0; db < DB; ++db) oacc[db] = mfma(vtf[cc][db], pb, oacc[db]);
    }
  }

  // the four waves' results meet:  O = sum_w 2^(m_w - m) O_w / sum_w 2^(m_w - m) l_w
  const float l_row = half_sum(l_run);
  if (h == 0) { stat_m[wave][c] = m_run; stat_l[wave][c] = l_row; }
  __syncthreads();   // (and every wave is done with its ring)
  float m = stat_m[0][c];
#pragma unroll
  for (int w = 1; w < 4; ++w) m = __builtin_fmaxf(m, stat_m[w][c]);
  float l = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) l += __builtin_amdgcn_exp2f(stat_m[w][c] - m) * stat_l[w][c];
  put_acc<D>(smem + wave * (kShortRows * D * 4), oacc, lane, __builtin_amdgcn_exp2f(m_run - m));
  __syncthreads();
  if (!row_valid) return;
  const float inv = 1.0f / l;
#pragma unroll
  for (int db = 0; db < DB; ++db) {
    const f32x4 x = sum_acc<D>(smem, (db * 4 + wave) * 64 + lane);   // wave w holds register quads rq = w
    *reinterpret_cast<uint2*>(o + ((size_t)my_row * Hq + head) * D + 32 * db + 8 * wave + 4 * h) =
        pack4(x[0] * inv, x[1] * inv, x[2] * inv, x[3] * inv);
  }
  if (wave == 0 && h == 0) lse[(size_t)head * N + my_row] = (m + __builtin_amdgcn_logf(l)) * kLn2;
}

// Backward.  The first `kv_blocks` workgroups take 32 keys and one q head each and sweep the query
// blocks from the diagonal to the document end; the others take 32 queries of one q head and sweep
// the key blocks up to the diagonal.  With grouped-query attention the first kind stores fp32
// [dK | dV] per q head, which bwd_short_group_kernel adds up: sweeping the heads of a group in one
// workgroup would make the longest chain g times as long (777 tokens, 8 q heads on 2 kv heads: 54 us).
template <int D>
__global__ void __launch_bounds__(kThreads, D == 64 ? 2 : 1)
bwd_short_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
                 const __bf16* __restrict__ o, const __bf16* __restrict__ d_o, const float* __restrict__ lse,
                 __bf16* __restrict__ dq, __bf16* __restrict__ dk, __bf16* __restrict__ dv, int Hq, int Hkv,
                 float scale, int kv_blocks, float* __restrict__ partials, PlanArgs plan) {
  constexpr int KK = D / 16, DB = D / 32;
  constexpr int kBlockBytes = kShortRows * D * 2;
  constexpr int kWaveBytes = 5 * kBlockBytes;      // two stages of Q and dO (K and V), one of O
  constexpr int kAccBytes = kShortRows * D * 4;
  // 160 KB at d = 128: all of a compute unit's LDS
  __shared__ __attribute__((aligned(1024))) char smem[4 * kWaveBytes];

  const int N = plan.N;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, c = lane & 31;
  const int bid = blockIdx.x;
  const float cs = scale * kLog2e;
  char* const ring = smem + wave * kWaveBytes;
  const unsigned lds = lds_addr_of(smem) + wave * kWaveBytes;
  const unsigned q_stride = (unsigned)((size_t)Hq * D * 2), kv_stride = (unsigned)((size_t)Hkv * D * 2);
  FragOffsets<D> fo;
  ShortTile it;
  int unit, head;

  if (bid >= kv_blocks) {
    // ---------------------------------------------------------------- dQ of 32 queries, one q head
    decode_block(bid - kv_blocks, Hq, unit, head);
    if (!derive_short_tile(plan, true, unit, true, lane, it)) return;
    const int kvh = head / (Hq / Hkv);
    const int my_row = it.row0 + c;
    const bool row_valid = my_row < it.doc_end;
    const int n_blocks = (it.row0 - it.doc_start) / kShortRows + 1;
    BlockLoader<D> loader;
    loader.init(lane, kv_stride);
    const unsigned long long step = 4ull * kShortRows * kv_stride;
    unsigned long long k_next = uniform64(k + ((size_t)(it.doc_start + kShortRows * wave) * Hkv + kvh) * D);
    unsigned long long v_next = uniform64(v + ((size_t)(it.doc_start + kShortRows * wave) * Hkv + kvh) * D);
    auto issue = [&](int block, int stage) __attribute__((always_inline)) {
      const int valid = it.doc_end - it.doc_start - kShortRows * block;
      loader.issue(k_next, valid, lds + stage * 2 * kBlockBytes);
      loader.issue(v_next, valid, lds + stage * 2 * kBlockBytes + kBlockBytes);
      k_next += step; v_next += step;
    };
    if (wave < n_blocks) issue(wave, 0);
    bf16x8 qf[KK], dof[KK];
    const int load_row = min(my_row, it.doc_end - 1);   // rows past the document end: duplicates, never stored
    const size_t row_off = ((size_t)load_row * Hq + head) * D;
    const float lse_row = lse[(size_t)head * N + load_row];
    float d_part = 0.f;
    {
      bf16x8 of[KK];
      load_row_frags<D>(d_o + row_off, h, dof);
      load_row_frags<D>(o + row_off, h, of);
      load_row_frags<D>(q + row_off, h, qf);
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) d_part = dot8(dof[kk], of[kk], d_part);
    }
    const float dsum = half_sum(d_part);
    const float lse2 = row_valid ? lse_row * kLog2e : 1e30f;
    fo.init(lane);
    wait_all_vm_visible();
    pin_frags(qf);
    pin_frags(dof);
    f32x16 acc[DB];
#pragma unroll
    for (int i = 0; i < DB; ++i) acc[i] = f32x16(0.f);
    int stage = 0;
#pragma unroll 1
    for (int j = wave; j < n_blocks; j += 4, stage ^= 1) {
      if (j + 4 < n_blocks) { issue(j + 4, stage ^ 1); wait_vm<2 * BlockLoader<D>::kInstr>(); }
      else wait_vm<0>();
      const char* kt = ring + stage * 2 * kBlockBytes;
      const char* vt = kt + kBlockBytes;
      f32x16 s, dp;
      bf16x8 kf[KK], vf[KK];
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) { kf[kk] = lds_read_frag(kt, fo.row_frag[kk]); vf[kk] = lds_read_frag(vt, fo.row_frag[kk]); }
      __builtin_amdgcn_sched_barrier(0);
      static_for<KK>([&](auto kk) __attribute__((always_inline)) {
        mfma_vgpr_acc<kk == 0>(s, kf[kk], qf[kk]);
        mfma_vgpr_acc<kk == 0>(dp, vf[kk], dof[kk]);
      });
      bf16x8 ktf[2][DB];
#pragma unroll
      for (int cc = 0; cc < 2; ++cc)
#pragma unroll
        for (int db = 0; db < DB; ++db) ktf[cc][db] = read_trans<D>(kt, fo, cc, db);
      mfma_vgpr_settle();
      if (j == n_blocks - 1) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (8 * (r / 4) + (r % 4) > c - 4 * h) s[r] = -INFINITY;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r)
        s[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], cs, -lse2)) * (dp[r] - dsum);
#pragma unroll
      for (int cc = 0; cc < 2; ++cc) {
        const bf16x8 dsb = pack8(s, 8 * cc);
#pragma unroll
        for (int db = 0; db < DB; ++db) acc[db] = mfma(ktf[cc][db], dsb, acc[db]);
      }
    }
    __syncthreads();   // every wave is done with its ring
    put_acc<D>(smem + wave * kAccBytes, acc, lane, scale);
    __syncthreads();
    if (!row_valid) return;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      const f32x4 x = sum_acc<D>(smem, (db * 4 + wave) * 64 + lane);
      *reinterpret_cast<uint2*>(dq + ((size_t)my_row * Hq + head) * D + 32 * db + 8 * wave + 4 * h) =
          pack4(x[0], x[1], x[2], x[3]);
    }
    return;
  }

  // ------------------------------------------------------------------ dK, dV of 32 keys, one q head
  decode_block(bid, Hq, unit, head);
  if (!derive_short_tile(plan, true, unit, false, lane, it)) return;
  const int kvh = head / (Hq / Hkv);
  const int my_kv = it.row0 + c;
  const bool kv_valid = my_kv < it.doc_end;
  const int n_blocks = (it.doc_end - it.row0 + kShortRows - 1) / kShortRows;   // the first one is the diagonal block
  BlockLoader<D> loader;
  loader.init(lane, q_stride);
  const unsigned long long step = 4ull * kShortRows * q_stride;
  const size_t first = ((size_t)(it.row0 + kShortRows * wave) * Hq + head) * D;
  unsigned long long q_next = uniform64(q + first), do_next = uniform64(d_o + first), o_next = uniform64(o + first);
  float lse_next = 0.f;
  auto rows_left = [&](int b) __attribute__((always_inline)) { return it.doc_end - it.row0 - kShortRows * b; };
  auto issue_qdo = [&](int b, int stage) __attribute__((always_inline)) {
    loader.issue(q_next, rows_left(b), lds + stage * 2 * kBlockBytes);
    loader.issue(do_next, rows_left(b), lds + stage * 2 * kBlockBytes + kBlockBytes);
    q_next += step; do_next += step;
  };
  auto issue_o = [&](int b) __attribute__((always_inline)) {
    loader.issue(o_next, rows_left(b), lds + 4 * kBlockBytes);
    o_next += step;
  };
  auto load_lse = [&](int b) __attribute__((always_inline)) {
    return lse[(size_t)head * N + min(it.row0 + kShortRows * b + c, it.doc_end - 1)];
  };
  if (wave < n_blocks) {
    lse_next = load_lse(wave);
    issue_qdo(wave, 0);
    issue_o(wave);
  }
  bf16x8 kf[KK], vf[KK];
  const size_t kv_off = ((size_t)min(my_kv, it.doc_end - 1) * Hkv + kvh) * D;
  load_row_frags<D>(k + kv_off, h, kf);
  load_row_frags<D>(v + kv_off, h, vf);
  fo.init(lane);
  wait_all_vm_visible();
  pin_frags(kf);
  pin_frags(vf);
  f32x16 dkacc[DB], dvacc[DB];
#pragma unroll
  for (int i = 0; i < DB; ++i) { dkacc[i] = f32x16(0.f); dvacc[i] = f32x16(0.f); }
  int stage = 0;
#pragma unroll 1
  for (int qb = wave; qb < n_blocks; qb += 4, stage ^= 1) {
    wait_vm<0>();
    const float lse2_row = lse_next * kLog2e;   // of query c, on lane c
    __builtin_amdgcn_sched_barrier(0);
    if (qb + 4 < n_blocks) {
      lse_next = load_lse(qb + 4);
      issue_qdo(qb + 4, stage ^ 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    const char* qt = ring + stage * 2 * kBlockBytes;
    const char* dot = qt + kBlockBytes;
    const char* ot = ring + 4 * kBlockBytes;
    // D, the statistics' way to the accumulator rows and the transposed fragments run behind the
    // matrix instructions of S and dP
    f32x16 s, dp;
    bf16x8 qa[KK], da[KK], of[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) { qa[kk] = lds_read_frag(qt, fo.row_frag[kk]); da[kk] = lds_read_frag(dot, fo.row_frag[kk]); }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) of[kk] = lds_read_frag(ot, fo.row_frag[kk]);
    __builtin_amdgcn_sched_barrier(0);
    float d_part = 0.f;
    static_for<KK>([&](auto kk) __attribute__((always_inline)) {
      mfma_vgpr_acc<kk == 0>(s, qa[kk], kf[kk]);
      mfma_vgpr_acc<kk == 0>(dp, da[kk], vf[kk]);
    });
    static_for<KK>([&](auto kk) __attribute__((always_inline)) { d_part = dot8(da[kk], of[kk], d_part); });
    const float d_row = half_sum(d_part);
    __builtin_amdgcn_sched_barrier(0);
    if (qb + 4 < n_blocks) issue_o(qb + 4);
    __builtin_amdgcn_sched_barrier(0);
    float lse_r[16], d_r[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int src = 8 * (r / 4) + (r % 4) + 4 * h;
      lse_r[r] = __shfl(lse2_row, src);
      d_r[r] = __shfl(d_row, src);
    }
    bf16x8 tq[2][DB], td[2][DB];
#pragma unroll
    for (int cc = 0; cc < 2; ++cc)
#pragma unroll
      for (int db = 0; db < DB; ++db) { td[cc][db] = read_trans<D>(dot, fo, cc, db); tq[cc][db] = read_trans<D>(qt, fo, cc, db); }
    mfma_vgpr_settle();
    const int q0 = it.row0 + kShortRows * qb;
    if (qb == 0 || q0 + kShortRows > it.doc_end) {   // wave-uniform
      const int t_lo = qb == 0 ? c - 4 * h : -64, t_hi = it.doc_end - q0 - 4 * h;   // allowed: t_lo <= 8 (r / 4) + r % 4 < t_hi
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int t = 8 * (r / 4) + (r % 4);
        if (t < t_lo || t >= t_hi) s[r] = -INFINITY;
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], cs, -lse_r[r]));
      dp[r] = s[r] * (dp[r] - d_r[r]);
    }
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
      const bf16x8 pb = pack8(s, 8 * cc), dsb = pack8(dp, 8 * cc);
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        dvacc[db] = mfma(td[cc][db], pb, dvacc[db]);
        dkacc[db] = mfma(tq[cc][db], dsb, dkacc[db]);
      }
    }
  }
  __syncthreads();   // every wave is done with its ring
  // dK of the four waves, then dV (both at once would not fit next to each other)
#pragma unroll
  for (int tensor = 0; tensor < 2; ++tensor) {
    if (tensor) __syncthreads();
    put_acc<D>(smem + wave * kAccBytes, tensor ? dvacc : dkacc, lane, tensor ? 1.0f : scale);
    __syncthreads();
    float* part = partials + (((size_t)unit * Hq + head) * 2 + tensor) * (kShortRows * D);
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      const int f4 = (db * 4 + wave) * 64 + lane;
      const f32x4 x = sum_acc<D>(smem, f4);
      if (Hq != Hkv) *reinterpret_cast<f32x4*>(part + f4 * 4) = x;
      else if (kv_valid)
        *reinterpret_cast<uint2*>((tensor ? dv : dk) + ((size_t)my_kv * Hkv + kvh) * D + 32 * db + 8 * wave + 4 * h) =
            pack4(x[0], x[1], x[2], x[3]);
    }
  }
}

// dK and dV of 32 keys and one kv head: the sum over the q heads of the group, in head order.
template <int D>
__global__ void __launch_bounds__(kThreads)
bwd_short_group_kernel(const float* __restrict__ partials, __bf16* __restrict__ dk, __bf16* __restrict__ dv,
                       int Hq, int Hkv, PlanArgs plan) {
  constexpr int DB = D / 32;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5, c = lane & 31;
  const int tensor = blockIdx.x & 1, kvh = (blockIdx.x >> 1) % Hkv, unit = (blockIdx.x >> 1) / Hkv;
  const int g = Hq / Hkv;
  ShortTile it;
  const float* p0 = partials + (((size_t)unit * Hq + kvh * g) * 2 + tensor) * (kShortRows * D) + threadIdx.x * 4;
  if (!derive_short_tile(plan, true, unit, false, lane, it)) return;
  f32x4 acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int j = 0; j < g; ++j)
#pragma unroll
    for (int db = 0; db < DB; ++db)
      acc[db] += *reinterpret_cast<const f32x4*>(p0 + (size_t)j * 2 * (kShortRows * D) + db * kThreads * 4);
  const int row = it.row0 + c;
  if (row >= it.doc_end) return;
#pragma unroll
  for (int db = 0; db < DB; ++db)
    *reinterpret_cast<uint2*>((tensor ? dv : dk) + ((size_t)row * Hkv + kvh) * D + 32 * db + 8 * wave + 4 * h) =
        pack4(acc[db][0], acc[db][1], acc[db][2], acc[db][3]);
}

}  // namespace

#endif  // VARLEN_ATTN_SHORT_HPP_
