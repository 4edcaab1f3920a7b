// Document-masked causal attention, forward and backward, for packed variable-length
// microbatches on MI355X (gfx950 / CDNA4).  Hand-written HIP; wave64; bf16 MFMA
// (v_mfma_f32_32x32x16_bf16) with fp32 accumulation.
//
// The operation is the quadratic term of the micro-batch time model (Section 5.2, Eq. 1):
// documents of lengths l_1..l_k packed into N tokens, block-diagonal mask, causal inside
// each block.  Only (query tile, key tile) pairs that contain an allowed (t, j) are ever
// visited, so the work follows sum l_i^2, not N^2.
//
// Sources: tiles.hpp (types, MFMA, LDS tile addressing and the register conventions),
// staging.hpp (direct-to-LDS loads), panels.hpp (what the kernels with one wave a SIMD share), plan.hpp,
// fragments.hpp (partial-result layout), fwd.hpp, fwd_wide.hpp (waves of 64 rows), bwd.hpp, bwd_pool.hpp (the
// backward as one pool of units), short.hpp (small microbatches in one launch each way); this file holds the
// profiler, the host side and the C ABI.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>
#include <utility>
#include <mutex>
#include <vector>

#include "varlen_attn.h"
#include "varlen_attn_bench.h"   // declares the event profiler exported from here

#include "tiles.hpp"
#include "staging.hpp"
#include "plan.hpp"
#include "fragments.hpp"
#include "fwd.hpp"
#include "fwd_wide.hpp"
#include "bwd.hpp"
#include "short.hpp"
#include "bwd_pool.hpp"

namespace {

// ----------------------------------------------------------------------------------------
// Optional per-kernel timing (host-side HIP events only; off by default).
// ----------------------------------------------------------------------------------------
enum KernelId {
  kPlan = 0, kFwd, kFwdCombine, kDq, kDkv, kBwdCombine, kPrep, kBwdPool, kBwdPoolCombine, kFusedBwd, kDqFinish, kFwdShort, kBwdShort,
  kBwdShortGroup, kFwdWide, kNumKernels
};
const char* const kKernelNames[kNumKernels] = {
    "plan_kernel", "fwd_kernel", "fwd_combine_kernel", "bwd_dq_kernel", "bwd_dkv_kernel",
    "bwd_combine_kernel", "bwd_prep_kernel", "bwd_pool_kernel", "bwd_pool_combine_kernel", "bwd_fused_kernel",
    "bwd_dq_finish_kernel", "fwd_short_kernel", "bwd_short_kernel", "bwd_short_group_kernel",
    "fwd_wide_kernel"};
struct Profiler {
  std::mutex mu;
  bool enabled = false;
  struct Rec { int id; hipEvent_t start, stop; };
  std::vector<Rec> recs;
  std::vector<hipEvent_t> pool;
  hipEvent_t get() {
    if (!pool.empty()) { hipEvent_t e = pool.back(); pool.pop_back(); return e; }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
  }
};
Profiler& profiler() { static Profiler p; return p; }

// Brackets one launch with events when profiling is on.
struct ScopedKernelTimer {
  hipStream_t stream; hipEvent_t stop = nullptr;
  ScopedKernelTimer(int id, hipStream_t s) : stream(s) {
    Profiler& p = profiler();
    if (!p.enabled) return;
    std::lock_guard<std::mutex> g(p.mu);
    hipEvent_t start = p.get();
    stop = p.get();
    if (!start || !stop) { stop = nullptr; return; }
    (void)hipEventRecord(start, stream);
    p.recs.push_back({id, start, stop});
  }
  ~ScopedKernelTimer() { if (stop) (void)hipEventRecord(stop, stream); }
};


inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

}  // namespace

// ----------------------------------------------------------------------------------------
// Workspace of varlen_attn_fwd_static: device memory that belongs to the library, so that the
// call needs no workspace from the caller and allocates nothing.  Every GPU this library runs
// on holds its own copy of the array, at its own address, until the process ends.  In host
// code the name below is only a handle for hipGetSymbolAddress: the address that kernels and
// copies use is the one that call returns for the current device, kept in StaticScratch.
// ----------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[VARLEN_ATTN_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
struct StaticScratch {
  std::mutex mu;
  void* ptr[kMaxDevices] = {};
};
// Device address of `scratch` on the current device (looked up once per device).
int static_scratch(void** out) {
  static StaticScratch st;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return VARLEN_ATTN_LAUNCH_FAILED;
  std::lock_guard<std::mutex> g(st.mu);
  if (!st.ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return VARLEN_ATTN_LAUNCH_FAILED;
    st.ptr[dev] = p;
  }
  *out = st.ptr[dev];
  return VARLEN_ATTN_OK;
}

bool params_ok(const varlen_attn_params* p) {
  if (!p) return false;
  if (p->total_tokens < 1 || p->num_docs < 1 || p->num_q_heads < 1 || p->num_kv_heads < 1) return false;
  if (p->num_q_heads % p->num_kv_heads) return false;
  if (!(p->softmax_scale > 0.f) || !(p->softmax_scale < 3.0e38f)) return false;
  return true;
}

// The list of the pooled backward's dQ units lies right in front of the dQ accumulator's offset (the forward, and with it
// varlen_attn_fwd_static, reaches up to the column partial results only).
inline size_t dq_list_bytes(const varlen_attn_workspace_layout& L) {
  return align_up(sizeof(varlen_attn_unit) * L.max_units + sizeof(varlen_attn_combine_item) * L.max_combine, 256);
}
inline size_t dq_list_offset(const varlen_attn_workspace_layout& L) { return L.dq_accumulator_offset - dq_list_bytes(L); }

// Capacities depend on the params only.  Slots: enough for kTargetUnits (unit, head) pairs,
// never more than 8 per tile; with grouped-query attention every column tile takes a slot.
bool layout_of(const varlen_attn_params* p, varlen_attn_workspace_layout* L, int* slots_cap) {
  if (!params_ok(p) || (p->head_dim != 64 && p->head_dim != 128)) return false;
  const long long tiles = (long long)p->total_tokens / kTile + p->num_docs;
  if (tiles > (1 << 24)) return false;
  const int Hq = p->num_q_heads, g = Hq / p->num_kv_heads;
  // every grid (units x heads, reduction blocks: tiles x heads x 2 tensors x 16) stays below 2^31
  if (tiles * Hq * 48 >= (1ll << 31)) return false;
  const long long cap = std::min<long long>((kTargetUnits + Hq - 1) / Hq, 8 * tiles);
  *slots_cap = (int)cap;
  L->max_units = (int)(tiles + cap);
  L->max_combine = (int)tiles;
  L->max_row_slots = (int)cap;
  L->max_col_slots = (int)(cap + (g > 1 ? tiles : 0));
  const size_t frag = (size_t)kTile * p->head_dim * sizeof(float);
  const size_t fwd_part = frag + 2 * kThreads * sizeof(float);
  size_t off = align_up(sizeof(varlen_attn_plan_header), 256);
  L->row_units_offset = off; off = align_up(off + sizeof(varlen_attn_unit) * L->max_units, 256);
  L->col_units_offset = off; off = align_up(off + sizeof(varlen_attn_unit) * L->max_units, 256);
  L->row_combine_offset = off; off = align_up(off + sizeof(varlen_attn_combine_item) * L->max_combine, 256);
  L->col_combine_offset = off; off = align_up(off + sizeof(varlen_attn_combine_item) * L->max_combine, 256);
  // -D = -rowsum(dO * O) [Hq, N], then -LSE / scale [Hq, N]
  L->dsum_offset = off; off = align_up(off + 2 * sizeof(float) * (size_t)Hq * p->total_tokens, 256);
  L->row_partials_offset = off; off = align_up(off + fwd_part * Hq * L->max_row_slots, 256);
  L->col_partials_offset = off; off = align_up(off + 2 * frag * Hq * L->max_col_slots, 256);
  // the pooled backward's dQ units and their reduction list
  off = align_up(off + dq_list_bytes(*L), 256);
  // fused backward: fp32 dQ accumulator [N, Hq, d]
  L->dq_accumulator_offset = off;
  if (p->flags & VARLEN_ATTN_FLAG_FUSED_BWD)
    off = align_up(off + sizeof(float) * (size_t)p->total_tokens * Hq * p->head_dim, 256);
  L->total_bytes = off;
  return true;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

int check_common(const varlen_attn_params* p, const void* const* ptrs, int n_ptrs, void* ws,
                 size_t ws_bytes, varlen_attn_workspace_layout* L, int* slots_cap) {
  if (!params_ok(p)) return VARLEN_ATTN_INVALID_ARG;
  for (int i = 0; i < n_ptrs; ++i)
    if (!ptrs[i]) return VARLEN_ATTN_INVALID_ARG;
  if (!ws) return VARLEN_ATTN_INVALID_ARG;
  if (p->head_dim != 64 && p->head_dim != 128) return VARLEN_ATTN_UNSUPPORTED;
  for (int i = 0; i < n_ptrs; ++i)
    if (!aligned16(ptrs[i])) return VARLEN_ATTN_UNSUPPORTED;
  if (!aligned16(ws)) return VARLEN_ATTN_UNSUPPORTED;
  if (!layout_of(p, L, slots_cap)) return VARLEN_ATTN_UNSUPPORTED;
  if (ws_bytes < L->total_bytes) return VARLEN_ATTN_WORKSPACE_TOO_SMALL;
  return VARLEN_ATTN_OK;
}

struct Regions {
  varlen_attn_plan_header* hdr;
  varlen_attn_unit *row_units, *col_units, *dq_units;
  varlen_attn_combine_item *row_comb, *col_comb, *dq_comb;
  float *dsum, *row_part, *col_part, *dq_acc;
};
Regions regions_of(char* ws, const varlen_attn_workspace_layout& L) {
  return Regions{reinterpret_cast<varlen_attn_plan_header*>(ws),
                 reinterpret_cast<varlen_attn_unit*>(ws + L.row_units_offset),
                 reinterpret_cast<varlen_attn_unit*>(ws + L.col_units_offset),
                 reinterpret_cast<varlen_attn_unit*>(ws + dq_list_offset(L)),
                 reinterpret_cast<varlen_attn_combine_item*>(ws + L.row_combine_offset),
                 reinterpret_cast<varlen_attn_combine_item*>(ws + L.col_combine_offset),
                 reinterpret_cast<varlen_attn_combine_item*>(ws + dq_list_offset(L) + sizeof(varlen_attn_unit) * L.max_units),
                 reinterpret_cast<float*>(ws + L.dsum_offset),
                 reinterpret_cast<float*>(ws + L.row_partials_offset),
                 reinterpret_cast<float*>(ws + L.col_partials_offset),
                 reinterpret_cast<float*>(ws + L.dq_accumulator_offset)};
}

// (tile, head) pairs at most; up to one round of workgroups their order does not matter
inline long long tile_heads(const varlen_attn_params* p) {
  return ((long long)p->total_tokens / kTile + p->num_docs) * p->num_q_heads;
}

bool pooled_backward(const varlen_attn_params* p);
bool wide_forward(const varlen_attn_params* p);

// Chunk lengths (plan.hpp).  Short chunks balance, long ones spare prologues and partial results; where the best length lies
// was measured by forcing it (230 microbatches of 1 K to 65 K tokens, 5 to 25 lengths each), and the two lines are fits to
// those times, one pair for each kernel.  Against one round of resident workgroups, or else 512 units, on the same microbatches
// (geometric means; slowest in brackets): forward 1.048 times as fast at heads of 128 (0.97), 1.049 at 64 (0.96); dQ at 64 1.031;
// the backward with column chunks so chosen 1.072 at 128 in the pool (0.96), 1.040 at 64 (0.97).  With grouped queries, chunk
// length and heads a unit together (130 microbatches, all combinations): 1.073 in the pool (0.98), 1.148 in two kernels at
// 128, 1.078 at 64 (0.99).  The best length of each single microbatch would add 1 to 3 %.
// A forward whose units just miss one round loses up to half: 19038 tokens in 14 documents, one head of 64, 38.0 us with 508
// units and 69.9 with 552, hence the exact count.  A unit that sweeps a group of 8 and outlasts the rest is what the line for the
// longest unit is there for: 20406 tokens, 8 q heads on one kv head, 1.54 times the best without it.
void chunk_rules(const varlen_attn_params* p, PlanArgs* a) {
  const bool grouped = p->num_q_heads > p->num_kv_heads, pooled = pooled_backward(p);
  const int resident = kResidentGroups / p->num_q_heads;
  constexpr float kSlot = 1.f / kTargetUnits;   // slopes: against what falls to one of kTargetUnits (unit, head) slots
  if (p->head_dim == 64) {
    a->rule[0] = ChunkRule{0.875f * kSlot, 3, 0.875f * kSlot, 3, resident, kMinChunkSteps};
  } else {
    // One wave a SIMD gains less from more units than fit one round: from 26 steps a slot on its chunks are 8 steps shorter than those of
    // waves of 32 rows (200 packs of ragged documents 1.005 times as fast as with their line).  Below, the same line: one of 1.1 x + 4 cut
    // documents of equal length just short of their end (8 of 1451 tokens and 946 more, 6 q heads: 50.3 / 57.6 us).
    a->rule[0] = ChunkRule{1.3125f * kSlot, 3, kSlot, wide_forward(p) ? 11.f : 19.f, resident, kMinChunkSteps + 1};
  }
  if (pooled) {
    // Heads of 64 go by the lines of 128 where queries are grouped (57 packs with more than two q heads a kv head, 33 with two;
    // 0.6, 0.8, 1.25 and 1.6 times the length: 0.96, 0.98, 0.94, 0.86 and 0.95, 0.98, 0.99, 0.93 times as fast; half or twice
    // the heads a unit: 0.95 and 0.55, 0.90 and 0.99; the best of each pack 1.014 and 1.010), by a longer one where they are
    // not (50 packs, the same lengths: 0.96, 0.99, 0.96, 0.91; best 1.005).
    a->rule[1] = grouped ? ChunkRule{2.5f * kSlot, 2, 1.6f * kSlot, 26, 0, 0}
                 : p->head_dim == 64 ? ChunkRule{3.75f * kSlot, 3, 2 * kSlot, 33, 0, 0} : ChunkRule{3 * kSlot, 3, 1.6f * kSlot, 27, 0, 0};
    a->sweep = SweepRule{0.75f, 128, 3 * kSlot, 200, 2.5f * kSlot, 32};
  } else if (p->head_dim == 64) {
    a->rule[1] = grouped ? ChunkRule{1.15f * kSlot, 2, kSlot, 18, 0, 0} : ChunkRule{1.15f * kSlot, 3, kSlot, 11, 0, 0};
    a->sweep = SweepRule{0.75f, 512, 0, 0, kSlot, 32};   // two workgroups share a compute unit: more units are wanted
  } else {
    a->rule[1] = ChunkRule{2.5f * kSlot, 2, kSlot, 18, 0, 0};
    a->sweep = SweepRule{1, 160, 0, 0, 2 * kSlot, 8};
  }
}

PlanArgs plan_args(const varlen_attn_params* p, const int32_t* cu, const Regions& R,
                   const varlen_attn_workspace_layout& L, int slots_cap, int32_t* status_copy) {
  PlanArgs a;
  a.cu = cu; a.B = p->num_docs; a.N = p->total_tokens; a.Hq = p->num_q_heads;
  a.g = p->num_q_heads / p->num_kv_heads;
  a.no_split = (p->flags & VARLEN_ATTN_FLAG_NO_SPLIT) ? 1 : 0;
  a.force_ch[0] = (p->flags >> 8) & 0xFF;
  a.force_ch[1] = (p->flags >> 16) & 0xFF;
  a.force_hpu = (p->flags >> 24) & 0xF;
  a.hdr = R.hdr; a.units[0] = R.row_units; a.units[1] = R.col_units; a.units[2] = R.dq_units;
  a.comb[0] = R.row_comb; a.comb[1] = R.col_comb; a.comb[2] = R.dq_comb;
  a.max_units = L.max_units; a.max_combine = L.max_combine;
  a.max_slots[0] = a.max_slots[2] = L.max_row_slots; a.max_slots[1] = L.max_col_slots; a.slots_cap = slots_cap;
  a.directions = pooled_backward(p) ? 3 : 2;
  a.longest_first = tile_heads(p) > kResidentGroups;
  chunk_rules(p, &a);
  a.status_copy = status_copy;
  return a;
}

// a microbatch with few documents and tiles is planned by a single wave (lower latency)
inline bool small_plan(const varlen_attn_params* p) {
  const long long tiles = (long long)p->total_tokens / kTile + p->num_docs;
  return !(p->flags & VARLEN_ATTN_FLAG_PLAN_LARGE) && p->num_docs <= 2 * kPlanThreadsSmall &&
         tiles <= 4 * kPlanThreadsSmall;
}
// ... and, smaller still, needs no plan launch in front of the forward: its workgroups work out
// their own units while one of them makes the plan (see fwd_kernel).  Every workgroup pays for that
// again, so it is worth it up to three rounds of workgroups.  Forward on a plan launch / here, 82
// microbatches of 3000 to 32000 tokens, 4 to 32 heads: 1.18 .. 1.00 from 800 to 1536 (tile, head)
// pairs (head size 64 1.19 .. 1.02), 1.05 .. 0.98 from 1700 to 2200.  Longest first as soon as the
// units may exceed one round, unless all of them are short: 10063 of 11918 tokens in one document, 8
// heads, 768 pairs, took 288 us in tile order and 263 us on a plan launch.
inline bool self_planned_forward(const varlen_attn_params* p) {
  const long long tiles = (long long)p->total_tokens / kTile + p->num_docs;
  return small_plan(p) && !(p->flags & VARLEN_ATTN_FLAG_PLAN_FIRST) && p->num_docs <= kSelfPlanDocs &&
         tiles <= kSelfPlanTiles && tile_heads(p) <= 3 * kResidentGroups;
}

// ... and the smallest microbatches take the kernels of short.hpp, forward and backward apart.  Their
// time follows the number of 32-row tiles (one workgroup each), hence the bound on rows (tokens x q
// heads), and the longest document, whose chain one workgroup walks alone.  The host does not know that
// length, so the bound on tokens is low enough for packs of which one document holds half to all of the
// tokens; it grows with the heads, because with few of them most of the GPU idles behind that document.
// Over 3300 such packs of 1000 to 10000 tokens, 2 to 64 documents, 1 to 16 q heads, the chunked kernels
// take at least 0.86 times as long as these inside the bounds (0.53 to 0.8 times beyond them: 10000
// tokens, most of them in one document, on one head).  Packs of ordinary documents (log-normal, 360 of
// them) gain 0.98 to 1.8 forward and 1.02 to 2.9 backward inside, which is why the bounds are not lower.
inline bool short_sizes(const varlen_attn_params* p, bool backward) {
  const bool wide = p->head_dim == 128, grouped = p->num_q_heads > p->num_kv_heads;
  const long long heads = p->num_q_heads;
  long long max_rows, max_tokens;
  if (!backward) {
    max_rows = wide ? 13000 : 30000;
    max_tokens = wide ? std::min(1024 + 1536 * heads, 3840ll) : 2048 + 3072 * heads;
  } else {
    max_rows = wide ? (grouped ? 8500 : 10000) : (grouped ? 18000 : 20000);
    max_tokens = wide ? (grouped ? 768 : 1280) + 512 * heads : 1536 + (grouped ? 384 : 512) * heads;
  }
  // few documents: one of them holds most of the tokens
  max_tokens = std::min(max_tokens, (wide ? 1536 : 2048) + 384ll * (p->num_docs - 1));
  return p->num_docs <= kSelfPlanDocs && p->total_tokens <= max_tokens && p->total_tokens * heads <= max_rows;
}
inline bool short_path(const varlen_attn_params* p, bool backward) {
  return !(p->flags & (VARLEN_ATTN_FLAG_NO_SPLIT | VARLEN_ATTN_FLAG_GENERAL)) && (p->flags >> 8) == 0 && short_sizes(p, backward);
}

// Backward beyond the small microbatches: dQ units and column units as one pool (bwd_pool.hpp) or in
// a kernel each.  The pool gains where chains differ in length and where the matrix pipe is the bound (one tail and
// one set of prologues instead of two; dQ chains whole); it pays for a pass over dO and O in front of it, which the two kernels
// do without.  Two kernels / pool, heads of 128:
//   documents of 128 tokens and more on average, or up to 24000 rows (tokens x q heads): 1.00 .. 1.38, 1.09 in the mean (150 packs
//   of 500 to 40000 tokens, 1 to 32 heads); of these only shorter documents, measured again: 0.92 .. 1.63, 1.21 in the mean (63 packs);
//   shorter ones, more rows: 0.91 .. 1.09, 0.97 in the mean;
//   more than two q heads a kv head, documents of 128 to 400 tokens on average: 1.04 .. 1.72, 1.14 in the mean (45 packs), up to
//   160000 rows; above, where the two kernels have column units enough that sweep whole groups, 0.85 .. 1.16 (13 packs).
// (The host does not know the longest document.  Documents of equal length are the pool's worst case inside the rule: 0.95 with
// 32 of 512 tokens, 4 heads; of up to 127 tokens 0.90 .. 1.38, 1.07 in the mean of 20 packs, where all chains are 1 or 2
// steps.)
// With VARLEN_ATTN_FLAG_NO_SPLIT a document's bits must not depend on what else is in the pack, hence neither may the
// route: there the heads alone decide.  With at most two q heads a kv head, 160 uncut packs: 0.98 .. 2.04, 1.52 in the mean, up
// to 24000 rows, 0.93 .. 1.86, 1.28 in the mean, up to 80000, and 0.87 .. 1.25, 0.98 in the mean, above.
// Heads of 64: the two kernels run two waves a SIMD, which hide each other's vector work (as long as the matrix instructions there) once there are
// units enough for both; below that the pool's one launch, whole dQ chains and single tail win.  Units cost the pool more, and
// their number goes with (document, q head) pairs, since each has a tile that it does not fill; documents of one length just
// above a multiple of 128 have the most for their rows, and chains that do not differ.  Two kernels / pool, on buffers that no
// cache holds and on resident ones (geometric mean of the two), 860 packs of 10000 to 112000 rows, half of them of equal or
// nearly equal documents, of 90 to 2500 tokens on average:
//   one q head a kv head, inside the rule 0.99 .. 1.42, 1.15 in the mean;  up to 50000 rows in more than 110 pairs 0.73 .. 1.21, 0.94 (216
//   documents of 130 tokens: 20.7 / 27.3 us);  more rows (other packs, most of them ragged) 0.73 .. 1.11, 0.93;
//   two q heads a kv head, inside 0.93 .. 1.29, 1.14;  more than 450 pairs 0.73 .. 1.18, 1.00;  more rows (other packs) 0.76 .. 1.13, 0.94;
//   more, inside 0.95 .. 1.26, 1.08;  more rows with 8 q heads on one kv head 0.84 .. 1.12, 1.00.
inline bool pooled_backward(const varlen_attn_params* p) {
  const bool many_to_one = p->num_q_heads > 2 * p->num_kv_heads;
  if (p->flags & VARLEN_ATTN_FLAG_NO_SPLIT) return p->head_dim == 128 && !many_to_one;
  const long long rows = (long long)p->total_tokens * p->num_q_heads, mean = p->total_tokens / p->num_docs;
  if (p->head_dim == 64) {
    if (p->flags & VARLEN_ATTN_FLAG_FUSED_BWD) return false;   // its chunks and heads a unit are those of the two kernels
    const bool grouped = p->num_q_heads > p->num_kv_heads;
    const long long max_rows = many_to_one ? (mean < 250 ? 75000 : p->num_q_heads > 4 * p->num_kv_heads ? 80000 : 110000) : grouped ? 90000 : 50000;
    if (!many_to_one && (long long)p->num_docs * p->num_q_heads > (grouped ? 450 : 110)) return false;
    return !short_sizes(p, true) && rows <= max_rows && mean >= (grouped ? 90 : 128);
  }
  return !short_sizes(p, true) && (rows <= 24000 || mean >= (many_to_one && rows > 160000 ? 400 : 128));
}

// Forward with heads of 128 in waves of 64 rows (fwd_wide.hpp): nothing covers a unit's first loads there, so chains have to be
// long, the more so where a workgroup slot sees many of them one after the other.  The host knows the mean length only, and packs
// of documents of one length have the shortest chains for it.  Waves of 32 rows / of 64, on buffers that no cache holds and on
// resident ones (geometric mean of the two), 760 packs of 60000 to 400000 rows, half of them of equal or nearly equal documents:
//   inside the rule 0.98 .. 1.12, 1.05 in the mean, up to 40000 tokens, and 0.96 .. 1.13, 1.06, above (one pack below: 98147 tokens in
//   85 equal documents, 4 heads, 229 / 255 us);
//   60000 to 90000 rows, 700 to 2000 tokens on average 0.91 .. 1.08, 1.00 and 1.02 in the mean;
//   90000 to 180000, 700 to 850: 0.96 .. 1.05, 1.00 and 1.02;  above, 700 to 1100: 0.90 .. 1.08, 0.97 and 1.03 (94317 tokens
//   in 109 equal documents, 4 heads, 175 / 196 us).
// Fewer rows: 0.91 .. 1.09, 1.02 in the mean of 33 (8192 tokens in 9 documents, 4 heads: 30.8 / 32.0 us; where the data stay in the
// cache between passes 31.9 / 30.6); documents of 50 to 700 tokens 0.93 .. 1.04, 0.98 in the mean of 70.  With
// VARLEN_ATTN_FLAG_NO_SPLIT a document's bits must not depend on the rest of the pack: 32 rows (0.93 .. 1.05 in 16 uncut packs).
inline bool wide_forward(const varlen_attn_params* p) {
  const long long rows = (long long)p->total_tokens * p->num_q_heads, mean = p->total_tokens / p->num_docs;
  if (p->head_dim != 128 || (p->flags & VARLEN_ATTN_FLAG_NO_SPLIT) || rows < 60000) return false;
  return mean >= (rows < 90000 ? 2000 : rows < 180000 ? 850 : 1100);
}

int launch_plan(const varlen_attn_params* p, const PlanArgs& a, hipStream_t stream) {
  ScopedKernelTimer timer(kPlan, stream);
  // A barrier costs less with fewer waves, a sweep over the tiles more.  Plan with 1024 / 512 / 256 threads: 8192 tokens in 205
  // documents 13.9 / 12.1 / 11.4 us, 32768 in 126 17.4 / 16.1 / 17.0, 131072 in one 23.2 / 24.2 / 29.5, 65536 in 1638
  // 25.3 / 28.7 / 37.6; whole calls on 29 packs of more than 64 documents 1 : 1.018 : 1.002.
  const long long tiles = (long long)p->total_tokens / kTile + p->num_docs;
  if (small_plan(p)) plan_kernel<kPlanThreadsSmall><<<1, kPlanThreadsSmall, 0, stream>>>(a);
  else if (p->flags & VARLEN_ATTN_FLAG_PLAN_LARGE || tiles > 768) plan_kernel<kPlanThreadsLarge><<<1, kPlanThreadsLarge, 0, stream>>>(a);
  else if (tiles > 320) plan_kernel<512><<<1, 512, 0, stream>>>(a);
  else plan_kernel<256><<<1, 256, 0, stream>>>(a);
  return hipGetLastError() == hipSuccess ? VARLEN_ATTN_OK : VARLEN_ATTN_LAUNCH_FAILED;
}

// Workgroups of a reduction launch at most: four per compute unit, which start within 1 us (the
// dispatcher starts about 1200 workgroups per us; 512, 1024 and 2048 measure the same).
constexpr int kCombineGroups = 1024;
constexpr int kPoolGroups = 256;   // one workgroup per compute unit

// self_plan: the forward launch makes the plan itself (no plan launch went before)
template <int D>
void launch_fwd(const varlen_attn_params* p, const void* q, const void* k, const void* v, void* o,
                float* lse, const Regions& R, const varlen_attn_workspace_layout& L,
                hipStream_t stream, const PlanArgs& args, bool self_plan) {
  const int N = p->total_tokens, Hq = p->num_q_heads, Hkv = p->num_kv_heads;
  if (short_path(p, false)) {
    ScopedKernelTimer timer(kFwdShort, stream);
    const int plan_block = self_plan ? 1 : 0;
    fwd_short_kernel<D><<<dim3(plan_block + grid_for(N / kShortRows + p->num_docs, Hq)), kThreads, 0, stream>>>(
        (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, (__bf16*)o, lse, Hq, Hkv, p->softmax_scale, plan_block, args);
    return;
  }
  const bool wide = D == 128 && wide_forward(p);
  if constexpr (D == 128) {
    if (wide) {
      ScopedKernelTimer timer(kFwdWide, stream);
      if (self_plan)
        fwd_wide_kernel<true><<<dim3(grid_for(L.max_units, Hq) + 1), 128, 0, stream>>>(
            (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, R.hdr, R.row_units, (__bf16*)o, lse,
            R.row_part, N, Hq, Hkv, p->softmax_scale, L.max_units, args);
      else
        fwd_wide_kernel<false><<<dim3(grid_for(L.max_units, Hq)), 128, 0, stream>>>(
            (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, R.hdr, R.row_units, (__bf16*)o, lse,
            R.row_part, N, Hq, Hkv, p->softmax_scale, L.max_units, PlanArgs{});
    }
  }
  if (!wide) {
    ScopedKernelTimer timer(kFwd, stream);
    if (self_plan)
      fwd_kernel<D, true><<<dim3(grid_for(L.max_units, Hq) + 1), kThreads, 0, stream>>>(
          (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, R.hdr, R.row_units, (__bf16*)o, lse,
          R.row_part, N, Hq, Hkv, p->softmax_scale, L.max_units, args);
    else
      fwd_kernel<D, false><<<dim3(grid_for(L.max_units, Hq)), kThreads, 0, stream>>>(
          (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, R.hdr, R.row_units, (__bf16*)o, lse,
          R.row_part, N, Hq, Hkv, p->softmax_scale, L.max_units, PlanArgs{});
  }
  if (!(p->flags & VARLEN_ATTN_FLAG_NO_SPLIT)) {
    ScopedKernelTimer timer(kFwdCombine, stream);
    const int cut_tiles = std::max(1, std::min(L.max_combine, L.max_row_slots / 2));   // see launch_bwd
    const long long pieces = (long long)cut_tiles * Hq * (D / 16);   // see fwd_combine_kernel
    fwd_combine_kernel<D><<<dim3((unsigned)std::min<long long>(pieces, kCombineGroups)), kThreads, 0, stream>>>(
        R.hdr, R.row_comb, cut_tiles, R.row_part, (__bf16*)o, lse, N, Hq);
  }
}

template <int D>
void launch_bwd(const varlen_attn_params* p, const void* q, const void* k, const void* v,
                const void* o, const float* lse, const void* d_o, void* dq, void* dk, void* dv,
                const Regions& R, const varlen_attn_workspace_layout& L, hipStream_t stream, const PlanArgs& args) {
  const int N = p->total_tokens, Hq = p->num_q_heads, Hkv = p->num_kv_heads;
  const float scale = p->softmax_scale;
  if (short_path(p, true)) {
    ScopedKernelTimer timer(kBwdShort, stream);
    const int tiles = N / kShortRows + p->num_docs;
    const unsigned blocks = grid_for(tiles, Hq);
    bwd_short_kernel<D><<<dim3(2 * blocks), kThreads, 0, stream>>>(
        (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, (const __bf16*)o, (const __bf16*)d_o, lse,
        (__bf16*)dq, (__bf16*)dk, (__bf16*)dv, Hq, Hkv, scale, (int)blocks, R.col_part, args);
    if (Hq != Hkv) {
      ScopedKernelTimer group_timer(kBwdShortGroup, stream);
      bwd_short_group_kernel<D><<<dim3((unsigned)tiles * Hkv * 2), kThreads, 0, stream>>>(
          R.col_part, (__bf16*)dk, (__bf16*)dv, Hq, Hkv, args);
    }
    return;
  }
  float* neg_lse = R.dsum + (size_t)Hq * N;
  const bool fused = (p->flags & VARLEN_ATTN_FLAG_FUSED_BWD) != 0;
  const bool split = !(p->flags & VARLEN_ATTN_FLAG_NO_SPLIT);
  // A cut chain has at least two chunks and all chunks of cut chains fit the slots, so at most
  // max_row_slots / 2 tiles are cut in either direction.
  const int cut_tiles = std::max(1, std::min(L.max_combine, L.max_row_slots / 2));
  const int col_items = Hq != Hkv ? L.max_combine : cut_tiles;   // grouped-query attention: every tile is summed over its group
  if (!fused && pooled_backward(p)) {
    int* const tickets = reinterpret_cast<int*>(reinterpret_cast<char*>(R.hdr) + kTicketsOffset);
    {
      ScopedKernelTimer timer(kPrep, stream);
      constexpr int kRowsPerBlock = kThreads / (D / 8);
      const long long rows = (long long)N * Hq;
      bwd_prep_kernel<D, false><<<dim3((unsigned)((rows + kRowsPerBlock - 1) / kRowsPerBlock)), kThreads, 0, stream>>>(
          (const __bf16*)o, (const __bf16*)d_o, lse, R.dsum, neg_lse, nullptr, tickets, N, Hq, scale);
    }
    {
      ScopedKernelTimer timer(kBwdPool, stream);   // dK, dV and dQ
      bwd_pool_kernel<D><<<dim3(kPoolGroups), kThreads, 0, stream>>>(
          BwdArgs<D>{(const __bf16*)q, (const __bf16*)k, (const __bf16*)v, (const __bf16*)d_o, neg_lse, R.dsum, R.hdr, R.col_units,
                     R.dq_units, R.row_units, (__bf16*)dq, (__bf16*)dk, (__bf16*)dv, R.col_part, R.row_part, N, Hq, Hkv, L.max_units, scale, tickets});
    }
    if (split || Hq != Hkv) {
      const int dq_items = split ? cut_tiles : 0;
      const long long pieces = (long long)col_items * Hkv * (D / 8) + (long long)dq_items * Hq * (D / 16);
      ScopedKernelTimer timer(kBwdPoolCombine, stream);
      bwd_pool_combine_kernel<D><<<dim3((unsigned)std::min<long long>(pieces, 2 * kCombineGroups)), kThreads, 0, stream>>>(
          R.hdr, R.col_comb, col_items, R.col_part, R.dq_comb, R.row_comb, dq_items, R.row_part, (__bf16*)dq, (__bf16*)dk, (__bf16*)dv, Hq, Hkv, scale);
    }
    return;
  }
  if (fused) {
    // -D = -rowsum(dO * O), -LSE / scale, and the dQ accumulator cleared
    ScopedKernelTimer timer(kPrep, stream);
    constexpr int kRowsPerBlock = kThreads / (D / 8);
    const long long rows = (long long)N * Hq;
    bwd_prep_kernel<D, true><<<dim3((unsigned)((rows + kRowsPerBlock - 1) / kRowsPerBlock)), kThreads, 0, stream>>>(
        (const __bf16*)o, (const __bf16*)d_o, lse, R.dsum, neg_lse, R.dq_acc, nullptr, N, Hq, scale);
  } else {
    // also writes -D = -rowsum(dO * O) and -LSE / scale, which the dK/dV kernel reads
    ScopedKernelTimer timer(kDq, stream);
    bwd_dq_kernel<D><<<dim3(grid_for(L.max_units, Hq)), kThreads, 0, stream>>>(
        (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, (const __bf16*)o, (const __bf16*)d_o,
        lse, R.dsum, neg_lse, R.hdr, R.row_units, (__bf16*)dq, R.row_part, N, Hq, Hkv, scale,
        L.max_units);
  }
  const unsigned unit_blocks = grid_for(L.max_units, Hq);
  if (fused) {
    // one kernel for dQ, dK and dV; dQ is summed in fp32 in the workspace and rounded afterwards
    ScopedKernelTimer timer(kFusedBwd, stream);
    auto launch = [&](auto kernel) {
      kernel<<<dim3(unit_blocks), kThreads, 0, stream>>>(
          (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, (const __bf16*)d_o, neg_lse, R.dsum, R.hdr,
          R.col_units, (__bf16*)dk, (__bf16*)dv, R.col_part, N, Hq, Hkv, scale, L.max_units,
          (int)unit_blocks, R.row_comb, L.max_combine, R.row_part, (__bf16*)dq, R.dq_acc);
    };
    bool halves = false;
    if constexpr (D == 128) {
      halves = pooled_backward(p);
      if (halves) launch(bwd_dkv_kernel<D, true, true>);
    }
    if (!halves) launch(bwd_dkv_kernel<D, true>);
  } else {
    // behind its units: one workgroup per (cut tile, q head) that sums the dQ partials
    const unsigned dq_blocks = split ? (unsigned)cut_tiles * Hq : 0u;
    ScopedKernelTimer timer(kDkv, stream);
    bwd_dkv_kernel<D, false><<<dim3(unit_blocks + dq_blocks), kThreads, 0, stream>>>(
        (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, (const __bf16*)d_o, neg_lse, R.dsum, R.hdr,
        R.col_units, (__bf16*)dk, (__bf16*)dv, R.col_part, N, Hq, Hkv, scale, L.max_units,
        (int)unit_blocks, R.row_comb, L.max_combine, R.row_part, (__bf16*)dq, nullptr);
  }
  if (fused) {
    const long long n8 = (long long)N * Hq * D / 8;
    ScopedKernelTimer timer(kDqFinish, stream);
    bwd_dq_finish_kernel<D><<<dim3((unsigned)((n8 + kThreads - 1) / kThreads)), kThreads, 0, stream>>>(
        R.dq_acc, (__bf16*)dq, n8, scale);
  }
  if (split || Hq != Hkv) {
    const long long pieces = (long long)col_items * Hkv * (D / 8);   // see bwd_combine_kernel
    ScopedKernelTimer timer(kBwdCombine, stream);
    bwd_combine_kernel<D><<<dim3((unsigned)std::min<long long>(pieces, kCombineGroups)), kThreads, 0, stream>>>(
        R.hdr, R.col_comb, col_items, R.col_part, (__bf16*)dk, (__bf16*)dv, Hq, Hkv, scale);
  }
}

}  // namespace

extern "C" {

size_t varlen_attn_workspace_bytes(const varlen_attn_params* params) {
  varlen_attn_workspace_layout L;
  int cap;
  if (!layout_of(params, &L, &cap)) return 0;
  return L.total_bytes;
}

int varlen_attn_workspace_regions(const varlen_attn_params* params,
                                  varlen_attn_workspace_layout* out) {
  if (!out || !params_ok(params)) return VARLEN_ATTN_INVALID_ARG;
  int cap;
  if (!layout_of(params, out, &cap)) return VARLEN_ATTN_UNSUPPORTED;
  return VARLEN_ATTN_OK;
}

int varlen_attn_plan(const varlen_attn_params* params, const int32_t* cu_seqlens, void* workspace,
                     size_t workspace_bytes, void* hip_stream) {
  varlen_attn_workspace_layout L;
  int cap;
  const void* ptrs[] = {cu_seqlens};
  const int rc = check_common(params, ptrs, 1, workspace, workspace_bytes, &L, &cap);
  if (rc != VARLEN_ATTN_OK) return rc;
  return launch_plan(params, plan_args(params, cu_seqlens, regions_of(static_cast<char*>(workspace), L), L, cap, nullptr),
                     static_cast<hipStream_t>(hip_stream));
}

int varlen_attn_fwd(const varlen_attn_params* params, const void* q, const void* k, const void* v,
                    const int32_t* cu_seqlens, void* o, float* lse, void* workspace,
                    size_t workspace_bytes, void* hip_stream) {
  varlen_attn_workspace_layout L;
  int cap;
  const void* ptrs[] = {q, k, v, cu_seqlens, o, lse};
  int rc = check_common(params, ptrs, 6, workspace, workspace_bytes, &L, &cap);
  if (rc != VARLEN_ATTN_OK) return rc;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const Regions R = regions_of(static_cast<char*>(workspace), L);
  const PlanArgs args = plan_args(params, cu_seqlens, R, L, cap, nullptr);
  bool self_plan = false;
  if (!(params->flags & VARLEN_ATTN_FLAG_REUSE_PLAN)) {
    self_plan = self_planned_forward(params);
    if (!self_plan) {
      rc = launch_plan(params, args, stream);
      if (rc != VARLEN_ATTN_OK) return rc;
    }
  }
  if (params->head_dim == 128) launch_fwd<128>(params, q, k, v, o, lse, R, L, stream, args, self_plan);
  else launch_fwd<64>(params, q, k, v, o, lse, R, L, stream, args, self_plan);
  return hipGetLastError() == hipSuccess ? VARLEN_ATTN_OK : VARLEN_ATTN_LAUNCH_FAILED;
}

int varlen_attn_fwd_static(const varlen_attn_params* params, const void* q, const void* k,
                           const void* v, const int32_t* cu_seqlens, void* o, float* lse,
                           int32_t* plan_status, void* hip_stream) {
  varlen_attn_workspace_layout L;
  int cap;
  void* ws = nullptr;
  const void* ptrs[] = {q, k, v, cu_seqlens, o, lse};
  // validate against a workspace of unlimited size first: bad arguments keep their own codes
  if (!params_ok(params)) return VARLEN_ATTN_INVALID_ARG;
  for (const void* ptr : ptrs)
    if (!ptr) return VARLEN_ATTN_INVALID_ARG;
  if (plan_status && (reinterpret_cast<uintptr_t>(plan_status) & 3)) return VARLEN_ATTN_UNSUPPORTED;
  if (params->head_dim != 64 && params->head_dim != 128) return VARLEN_ATTN_UNSUPPORTED;
  for (const void* ptr : ptrs)
    if (!aligned16(ptr)) return VARLEN_ATTN_UNSUPPORTED;
  if (!layout_of(params, &L, &cap)) return VARLEN_ATTN_UNSUPPORTED;
  // the forward touches the workspace up to the end of the row partial results only
  if (L.col_partials_offset > (size_t)VARLEN_ATTN_STATIC_SCRATCH_BYTES) return VARLEN_ATTN_STATIC_TOO_LARGE;
  int rc = static_scratch(&ws);
  if (rc != VARLEN_ATTN_OK) return rc;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const Regions R = regions_of(static_cast<char*>(ws), L);
  PlanArgs args = plan_args(params, cu_seqlens, R, L, cap, plan_status);
  // No backward follows (and the array ends in front of a third list).  The short kernels take their tiles from the documents: only
  // the status word is wanted (889 tokens in one document, 16 q heads of 64: 8.2 us, 8.5 with a plan that nobody reads).
  args.directions = short_path(params, false) ? 0 : 1;
  const bool self_plan = self_planned_forward(params);
  if (!self_plan) rc = launch_plan(params, args, stream);
  if (rc != VARLEN_ATTN_OK) return rc;
  if (params->head_dim == 128) launch_fwd<128>(params, q, k, v, o, lse, R, L, stream, args, self_plan);
  else launch_fwd<64>(params, q, k, v, o, lse, R, L, stream, args, self_plan);
  return hipGetLastError() == hipSuccess ? VARLEN_ATTN_OK : VARLEN_ATTN_LAUNCH_FAILED;
}

int varlen_attn_bwd(const varlen_attn_params* params, const void* q, const void* k, const void* v,
                    const void* o, const float* lse, const void* d_o, const int32_t* cu_seqlens,
                    void* dq, void* dk, void* dv, void* workspace, size_t workspace_bytes,
                    void* hip_stream) {
  varlen_attn_workspace_layout L;
  int cap;
  const void* ptrs[] = {q, k, v, o, lse, d_o, cu_seqlens, dq, dk, dv};
  int rc = check_common(params, ptrs, 10, workspace, workspace_bytes, &L, &cap);
  if (rc != VARLEN_ATTN_OK) return rc;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const Regions R = regions_of(static_cast<char*>(workspace), L);
  const PlanArgs args = plan_args(params, cu_seqlens, R, L, cap, nullptr);
  if (!(params->flags & VARLEN_ATTN_FLAG_REUSE_PLAN)) {
    rc = launch_plan(params, args, stream);
    if (rc != VARLEN_ATTN_OK) return rc;
  }
  if (params->head_dim == 128) launch_bwd<128>(params, q, k, v, o, lse, d_o, dq, dk, dv, R, L, stream, args);
  else launch_bwd<64>(params, q, k, v, o, lse, d_o, dq, dk, dv, R, L, stream, args);
  return hipGetLastError() == hipSuccess ? VARLEN_ATTN_OK : VARLEN_ATTN_LAUNCH_FAILED;
}

int varlen_attn_check(const void* workspace, void* hip_stream) {
  if (!workspace) return VARLEN_ATTN_INVALID_ARG;
  varlen_attn_plan_header hdr;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (hipMemcpyAsync(&hdr, workspace, sizeof(hdr), hipMemcpyDeviceToHost, stream) != hipSuccess)
    return VARLEN_ATTN_LAUNCH_FAILED;
  if (hipStreamSynchronize(stream) != hipSuccess) return VARLEN_ATTN_LAUNCH_FAILED;
  return hdr.status;
}

int varlen_attn_profile(int enable) {
  Profiler& p = profiler();
  std::lock_guard<std::mutex> g(p.mu);
  for (auto& r : p.recs) { p.pool.push_back(r.start); p.pool.push_back(r.stop); }
  p.recs.clear();
  p.enabled = enable != 0;
  return VARLEN_ATTN_OK;
}

int varlen_attn_profile_read(varlen_attn_kernel_time* out, int capacity) {
  if (!out || capacity < 1) return VARLEN_ATTN_INVALID_ARG;
  Profiler& p = profiler();
  std::lock_guard<std::mutex> g(p.mu);
  float total[kNumKernels] = {0};
  int count[kNumKernels] = {0};
  for (auto& r : p.recs) {
    float ms = 0.f;
    if (hipEventSynchronize(r.stop) != hipSuccess || hipEventElapsedTime(&ms, r.start, r.stop) != hipSuccess)
      return VARLEN_ATTN_LAUNCH_FAILED;
    total[r.id] += ms;
    count[r.id] += 1;
    p.pool.push_back(r.start);
    p.pool.push_back(r.stop);
  }
  p.recs.clear();
  int n = 0;
  for (int i = 0; i < kNumKernels && n < capacity; ++i) {
    if (!count[i]) continue;
    out[n].name = kKernelNames[i];
    out[n].launches = count[i];
    out[n].total_ms = total[i];
    ++n;
  }
  return n;
}

const char* varlen_attn_status_string(int status) {
  switch (status) {
    case VARLEN_ATTN_OK: return "ok";
    case VARLEN_ATTN_INVALID_ARG: return "invalid argument";
    case VARLEN_ATTN_UNSUPPORTED: return "unsupported head_dim or misaligned pointer";
    case VARLEN_ATTN_WORKSPACE_TOO_SMALL: return "workspace too small";
    case VARLEN_ATTN_LAUNCH_FAILED: return "kernel launch failed";
    case VARLEN_ATTN_BAD_CU_SEQLENS: return "malformed cu_seqlens";
    case VARLEN_ATTN_PLAN_OVERFLOW: return "plan does not fit the workspace";
    case VARLEN_ATTN_STATIC_TOO_LARGE: return "problem exceeds the library's static workspace";
    default: return "unknown status";
  }
}

}  // extern "C"
