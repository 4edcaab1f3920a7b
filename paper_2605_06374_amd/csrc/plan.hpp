// Plan kernel: cu_seqlens -> validated, chunked work units (integer work only).
#ifndef VARLEN_ATTN_PLAN_HPP_
#define VARLEN_ATTN_PLAN_HPP_

#include "tiles.hpp"

namespace {

// ----------------------------------------------------------------------------------------
// Plan: cu_seqlens -> validated work units (integer work only).
//
// One workgroup.  For both directions (0: row chains for forward / dQ, 1: column chains for
// dK / dV) it picks the chunk length, cuts every tile's chain into nearly equal chunks and
// writes the units.  Chunk length: at least kMinChunkSteps, by two lines in the microbatch's steps
// (ChunkRule), and always such that the partial-result slots fit the workspace.
//
// Units are placed longest first by cost class (kPlanClasses classes of equal width over the
// chunk lengths that occur): the hardware hands workgroups out in index order, so this is
// longest-job-first list scheduling.  The order inside a class is not defined.
//
// The kernel runs once per microbatch on a single compute unit, in front of everything else,
// so its latency is what counts: one thread per document, then one thread per tile (found by
// bisection in the running tile count of the documents), class counters per wave in LDS so that
// the same-address atomics of a wave stay inside the wave, and two sweeps over the tiles
// (count, then place) that run the same code.
// ----------------------------------------------------------------------------------------
constexpr int kPlanThreadsLarge = 1024;   // general form (also built for 256 and 512: launch_plan)
constexpr int kPlanThreadsSmall = 64;     // one wave: every barrier is free, nothing is shared between waves
constexpr int kPlanClasses = 32;
constexpr int kMinChunkSteps = 4;
constexpr int kResidentGroups = 512;  // 256 CUs x 2 workgroups (forward, dQ)
constexpr int kTargetUnits = 512;   // (unit, head) slots that chunk lengths are counted in and that cut chains may take
constexpr int kNoSplitSteps = 1 << 28;

// Behind the header the plan of at most kSelfPlanDocs documents and 65535 tokens keeps the documents'
// ends, so that the kernels that take their tiles from the documents themselves (short.hpp) need
// nothing but the plan either: a caller may refill cu_seqlens once the plan is made.  All zero, which
// is no partition of N tokens, when nothing was planned.
constexpr int kSelfPlanDocs = 64, kSelfPlanTiles = 256;
// ... and behind them the ticket counters of a backward (bwd_pool.hpp).
constexpr int kTicketsOffset = 192, kTicketCounters = 8;
static_assert(sizeof(varlen_attn_plan_header) + 2 * kSelfPlanDocs <= kTicketsOffset && kTicketsOffset + 4 * kTicketCounters <= 256,
              "the unit arrays start at byte 256");
__device__ __forceinline__ uint16_t* kept_ends(const varlen_attn_plan_header* hdr) {
  return reinterpret_cast<uint16_t*>(const_cast<varlen_attn_plan_header*>(hdr) + 1);
}

// Chunk length of a chain: ceil(slope * x) + base steps, or with slope2 and base2 where that is less (x: steps * Hq, what all
// heads' chains have together), kMinChunkSteps at least.  The lines are fits to measured times; the host picks
// them (chunk_rules() in varlen_attn.hip).  With `resident` units of a head that the GPU holds at once, 7/10 to 7/5 of that
// length, `shortest` at least, where it takes all units into one round.
struct ChunkRule { float slope, base, slope2, base2; int resident, shortest; };
// Grouped-query attention: chunks of column units that sweep h q heads are h^-power as long, and h is the largest that leaves
// min_units + min(units * x, max_units) units and none of more than slope * x + base (step, head) pairs.
struct SweepRule { float power, min_units, units, max_units, slope, base; };

// What every workgroup of a small microbatch reads comes first: behind the rules, 72 bytes into the kernel's arguments further on, it took
// 0.15 us longer (1402 tokens, 8 heads of 64, forward 8.84 -> 8.70 us).
struct PlanArgs {
  const int32_t* cu;
  int B, N, Hq, g, no_split;
  int force_ch[2];  // > 0: chunk length given by the caller (tuning), per direction
  int force_hpu;    // > 0: q heads per column unit given by the caller (a divisor of g)
  varlen_attn_plan_header* hdr;
  varlen_attn_unit* units[3];            // row units, column units, dQ units
  varlen_attn_combine_item* comb[3];
  int max_units, max_combine, max_slots[3], slots_cap;
  int directions;         // 0: status word only; 1: row units; 2: and column units; 3: and dQ units of their own chunk length
  bool longest_first;     // order in which the forward's workgroups take their own units (derive_row_unit)
  int32_t* status_copy;   // optional second place for the status word (device), or null
  ChunkRule rule[2];      // row chains, column chains
  SweepRule sweep;
};

// inclusive sum over the lanes of a wave: data-parallel-primitive moves (shifts inside rows of
// 16 lanes, then the last lane of a row broadcast into the rows behind it), which cost a vector
// instruction each where a shuffle goes through the LDS crossbar and back
template <int kCtrl, int kRowMask>
__device__ __forceinline__ int dpp_or_zero(int v) {
  return __builtin_amdgcn_update_dpp(0, v, kCtrl, kRowMask, 0xF, false);
}
__device__ __forceinline__ int wave_inclusive_sum(int v) {
  v += dpp_or_zero<0x111, 0xF>(v);   // row_shr:1
  v += dpp_or_zero<0x112, 0xF>(v);   // row_shr:2
  v += dpp_or_zero<0x114, 0xF>(v);   // row_shr:4
  v += dpp_or_zero<0x118, 0xF>(v);   // row_shr:8
  v += dpp_or_zero<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp_or_zero<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
  return v;
}
// value of lane `src` (wave-uniform) in every lane
__device__ __forceinline__ int lane_value(int v, int src) {
  return __builtin_amdgcn_readlane(v, __builtin_amdgcn_readfirstlane(src));
}

// Chunk length of a direction (ChunkRule).  `tries` > 0 tells that the units are to be resident at once: after each but the
// last that missed it the length may grow, up to 7/5 of the line's (`line`), and is the line's in the end.  In single
// precision without contraction: the forward workgroups of a small microbatch, whose steps are few enough to be exact, work it out
// for themselves and have to agree with the plan.
__device__ __forceinline__ int plan_chunk_steps(const ChunkRule& r, float steps, int n_tiles, int Hq, int forced, int& line,
                                                int& tries) {
#pragma clang fp contract(off)
  const float x = steps * (float)Hq;
  line = (int)min(max(min(ceilf(x * r.slope) + r.base, ceilf(x * r.slope2) + r.base2), (float)kMinChunkSteps), (float)kNoSplitSteps);
  tries = 0;
  if (forced > 0) return line = forced;
  if (n_tiles > r.resident || r.resident == 0) return line;
  // units of one head ~ steps / chunk + tiles / 2 (a cut chain rarely divides evenly)
  const float room = (float)(2 * r.resident - n_tiles);
  const int fill = max(max(r.shortest, (7 * line + 9) / 10), (int)ceilf(2.f * steps * __builtin_amdgcn_rcpf(room)));
  tries = 5 * fill <= 7 * line ? 2 : 0;
  return tries ? fill : line;
}

// The next chunk length when there are more chunks than `room` for them: longer in proportion, but by a sixteenth at least
// (every turn counts all chunks again) and at most twice as long.
__device__ __forceinline__ int longer_chunk(int ch, int chunks, int room) {
  const float more = (float)ch * (float)(chunks - room) * __builtin_amdgcn_rcpf((float)room);
  return ch + min(ch, max(1 + ch / 16, (int)min(more, (float)ch)));
}

// Chunks of at most `ch` steps over one document's chains, without a look at its tiles: `all` of them, `cut` in chains of more
// than one.  Chains 1 .. M have 2 t steps (2 t - 1 where `odd`), so every ch chains have one chunk each up to h of them, two
// up to ch, and 2 more than their predecessors ch before.
template <typename Int>
__device__ __forceinline__ void count_chunks(int M, int ch, bool odd, Int& all, Int& cut) {
  const Int h = (ch + (odd ? 1 : 0)) / 2, q = (unsigned)M / (unsigned)ch, r = (Int)M - q * ch;
  const Int chunks = ch * q * (q - 1) + q * (2 * (Int)ch - h) + 2 * q * r + r + max((Int)0, r - h);
  all += chunks;
  cut += chunks - min((Int)M, h);
}
// rows of a document of T tiles and S steps: T - 1 chains of 2 t steps and one of S
template <typename Int>
__device__ __forceinline__ void count_row_chunks(int T, int S, int ch, Int& all, Int& cut) {
  if (T <= 0) return;
  count_chunks<Int>(T - 1, ch, false, all, cut);
  const int last = (int)(((unsigned)S + (unsigned)ch - 1) / (unsigned)ch);
  all += last;
  cut += last > 1 ? last : 0;
}
// columns: T chains of S, S - 2, ... steps
template <typename Int>
__device__ __forceinline__ void count_col_chunks(int T, int S, int ch, Int& all, Int& cut) {
  if (T > 0) count_chunks<Int>(T, ch, S & 1, all, cut);
}

// At most `room` chunks of `ch` steps, without a count?  A chain of n steps has fewer than n / ch + 1.
__device__ __forceinline__ bool surely_fits(float steps, int n_tiles, int ch, int room) {
  return steps * __builtin_amdgcn_rcpf((float)ch) + 0.01f <= (float)(room - n_tiles);
}

// Another turn with a longer chunk?  `cut` chunks of cut chains have `slots`, `all` units one round of `resident`.
__device__ __forceinline__ bool next_chunk(int& ch, int line, int& tries, float steps, int cut, int slots, int all, int resident) {
#pragma clang fp contract(off)
  if (tries && all > resident) {
    // what is not in proportion to 1 / ch (chains that do not divide evenly) stays
    const float stays = (float)all - steps * __builtin_amdgcn_rcpf((float)ch), room = (float)resident - stays;
    const float longer = room > 0.f ? ceilf(min(steps * __builtin_amdgcn_rcpf(room), 1e6f)) + 1.f : 1e6f;
    if (--tries && longer * 5.f <= (float)(7 * line)) ch = max(ch + 1, (int)longer);
    else { tries = 0; ch = line; }
    return true;
  }
  if (cut <= slots) return false;
  ch = longer_chunk(ch, cut, slots);
  return true;
}

// Chunk length of a dQ with units of its own: the backward's resident workgroups draw column units and dQ units from one
// pool, so that a chain is cut only where it would outlast the rest: half of a workgroup's share, a column step
// counted as two (it takes 1.9 times as long).  From about 77 million tokens in one document the share is beyond 31 bits; it
// has the bound of a ChunkRule's lines (a chunk length below 1 would divide by zero where chains are cut).
__host__ __device__ __forceinline__ int plan_dq_steps(const unsigned long long* steps, int Hq, int row_steps, int forced) {
  if (forced > 0) return forced;
  const unsigned long long share = ((steps[0] + 2 * steps[1]) * Hq + kTargetUnits - 1) / kTargetUnits;
  return share >= (unsigned long long)kNoSplitSteps ? kNoSplitSteps : (int)share > row_steps ? (int)share : row_steps;
}

// ... and no shorter than this: with few steps a workgroup, what a cut costs (first loads, partial results, their sum) outweighs the
// balance.  Backward of 60 packs with heads of 128 (0.4 to 12 steps a slot), every chunk length forced: 0.973 of the time without it in the
// mean, 0.87 .. 1.05.  2 x + 10 steps take 0.978, 14 steps everywhere 0.976 (but 1.15 on packs of less than one step a slot).
__host__ __device__ __forceinline__ int plan_dq_shortest(unsigned long long row_steps, int Hq) {
  const float steps = 4.f * (1.f / kTargetUnits) * (float)row_steps * (float)Hq + 6.f;
  return steps < 16.f ? (int)steps : 16;
}

// sum, maximum and 64-bit sum over the lanes of a wave (all lanes get it)
__device__ __forceinline__ int wave_total(int v) { return lane_value(wave_inclusive_sum(v), 63); }
__device__ __forceinline__ int wave_max(int v) {   // v >= 0
  v = max(v, dpp_or_zero<0x111, 0xF>(v));
  v = max(v, dpp_or_zero<0x112, 0xF>(v));
  v = max(v, dpp_or_zero<0x114, 0xF>(v));
  v = max(v, dpp_or_zero<0x118, 0xF>(v));
  v = max(v, dpp_or_zero<0x142, 0xA>(v));
  v = max(v, dpp_or_zero<0x143, 0xC>(v));
  return lane_value(v, 63);
}
__device__ __forceinline__ unsigned long long wave_total_wide(unsigned long long v) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) v += __shfl_xor(v, off);
  return v;
}

// ----------------------------------------------------------------------------------------
// The u-th row unit of a microbatch of at most 64 documents and 256 tiles, in the order (tile, chunk) or, `longest_first`,
// (chunk length of the tile, tile, chunk), worked out by one wave from cu_seqlens alone with the plan's own rules (chunk
// length, nearly equal chunks, slots of cut tiles numbered in tile order): a forward workgroup of a small microbatch finds its
// unit this way instead of waiting for the plan.  All 64 lanes must call it; every lane gets the same answer.  False:
// cu_seqlens is malformed (the plan reports it) or u is past the last unit.
// ----------------------------------------------------------------------------------------
__device__ __forceinline__ bool derive_row_unit(const int32_t* __restrict__ cu, int B, int N, int Hq,
                                                int no_split, const ChunkRule& rule, int forced, int slots_cap, int u,
                                                bool longest_first, int lane, varlen_attn_unit& out) {
  int s = 0, e = 0;
  if (lane < B) { s = cu[lane]; e = cu[lane + 1]; }
  const int l = e - s;
  const int cu_first = lane_value(s, 0), cu_last = lane_value(e, B - 1);
  if (__any(lane < B && l < 0) || cu_first != 0 || cu_last != N) return false;
  const int T = (l + kTile - 1) / kTile, S = (l + kStep - 1) / kStep;
  const int t_incl = wave_inclusive_sum(T);   // tiles up to and including this document
  const int n_tiles = lane_value(t_incl, 63);
  const int steps = wave_total(T * (T - 1) + S);
  int ch = kNoSplitSteps, line = 0;
  int tries = 0;
  if (!no_split) ch = plan_chunk_steps(rule, (float)steps, n_tiles, Hq, forced, line, tries);
  constexpr int kRounds = kSelfPlanTiles / 64;
  static_assert(kRounds == 4, "chain lengths of four tiles a lane");
  int ds[kRounds], de[kRounds], row0[kRounds], n[kRounds], nc[kRounds];
  // tiles 64 r + lane: their document (the first whose running tile count exceeds the tile
  // index, found by bisection over the lanes), first row and chain length
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    ds[r] = de[r] = row0[r] = n[r] = 0;
    if (64 * r < n_tiles) {
      const int t = 64 * r + lane;
      // doc = number of documents whose running tile count is <= t (it is non-decreasing over
      // the lanes, and lane 63 holds n_tiles > t for every tile that exists)
      int doc = 0;
#pragma unroll
      for (int step = 32; step >= 1; step >>= 1)
        if (__shfl(t_incl, doc + step - 1) <= t) doc += step;
      ds[r] = __shfl(s, doc); de[r] = __shfl(e, doc);
      const int before = __shfl(t_incl - T, doc);
      row0[r] = ds[r] + (t - before) * kTile;
      n[r] = t < n_tiles ? (min(row0[r] + kTile, de[r]) - 1 - ds[r]) / kStep + 1 : 0;
    }
  }
  // the chunk length grows until the chunks of cut chains fit their slots
  bool again = !no_split && !surely_fits((float)steps, n_tiles, ch, tries ? min(slots_cap, rule.resident) : slots_cap);
#pragma unroll 1
  while (again) {
    int cut = 0, all = 0;
    count_row_chunks<int>(T, S, ch, all, cut);
    again = next_chunk(ch, line, tries, (float)steps, wave_total(cut), slots_cap, tries ? wave_total(all) : 0, rule.resident);
  }
#pragma unroll
  for (int r = 0; r < kRounds; ++r) nc[r] = n[r] ? (n[r] + ch - 1) / ch : 0;
  // Longest first: the units of tiles with chunks longer than x come before all others, F(x) of them.
  // The smallest x with F(x) <= u, found bit by bit, is the length of the unit asked for; among the
  // tiles of that length it is number u - F(x) in tile order.  One sum over the wave per bit of the
  // longest chunk; with none longer than kMinChunkSteps the order is worth less than finding it (760
  // tokens in 40 documents, 32 q heads: 20.9 us in tile order, 24.4 us with ten sums in every workgroup).
  int in_order[kRounds];   // units of the tile that count towards u
#pragma unroll
  for (int r = 0; r < kRounds; ++r) in_order[r] = nc[r];
  if (longest_first && ch > kMinChunkSteps && __any(max(max(n[0], n[1]), max(n[2], n[3])) > kMinChunkSteps)) {
    int len[kRounds], longest = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      len[r] = nc[r] ? (n[r] + nc[r] - 1) / nc[r] : 0;
      longest = max(longest, len[r]);
    }
    int bit = kSelfPlanTiles * kTile / kStep, before = 0;   // no chain has twice as many steps
    while (!__any(longest >= bit)) bit >>= 1;               // down to the top bit of the longest
    int x = 2 * bit - 1;
#pragma unroll 1
    for (; bit; bit >>= 1) {
      int longer = 0;
#pragma unroll
      for (int r = 0; r < kRounds; ++r) longer += len[r] > x - bit ? nc[r] : 0;
      longer = wave_total(longer);
      if (longer <= u) { x -= bit; before = longer; }
    }
    if (x == 0) return false;   // all units come before u
    u -= before;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) in_order[r] = len[r] == x ? nc[r] : 0;
  }
  int units_before = 0, slots_before = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    if (64 * r < n_tiles) {
      const int cut = nc[r] > 1 ? nc[r] : 0;
      const int u_incl = wave_inclusive_sum(in_order[r]), s_incl = wave_inclusive_sum(cut);
      const int u0 = units_before + u_incl - in_order[r];
      const unsigned long long hit = __ballot(u0 <= u && u < u0 + in_order[r]);
      if (hit) {
        const int src = __ffsll((long long)hit) - 1;
        const int nn = lane_value(n[r], src), k = lane_value(nc[r], src), c = u - lane_value(u0, src);
        const int slot0 = slots_before + lane_value(s_incl - cut, src);
        const int base = nn / k, rem = nn % k;
        const int first = c * base + min(c, rem), len = base + (c < rem ? 1 : 0);
        out = varlen_attn_unit{lane_value(row0[r], src), lane_value(ds[r], src), lane_value(de[r], src), first,
                               first + len, k > 1 ? slot0 + c : -1, len, 0};
        return true;
      }
      units_before += lane_value(u_incl, 63);
      slots_before += lane_value(s_incl, 63);
    }
  }
  return false;
}

template <int kPlanThreads>
__device__ __forceinline__ void plan_body(const PlanArgs& a) {
  constexpr int kPlanWaves = kPlanThreads / 64;
  // one wave: the tiles are visited in order, so the slots of cut row chains can be numbered in
  // tile order by a running sum (a forward workgroup that works out its own unit needs that)
  constexpr bool kOrdered = kPlanWaves == 1;
  static_assert(2 * kPlanClasses * kPlanWaves == kPlanThreads, "one thread per class counter");
  __shared__ int doc_first_tile[kPlanThreads + 1];  // running tile count of the batch's documents
  __shared__ int doc_s[kPlanThreads], doc_e[kPlanThreads];
  __shared__ int hist[3][kPlanClasses][kPlanWaves];    // units per (direction, class, wave), then cursors
  __shared__ int class_total[3][kPlanClasses];
  __shared__ int wave_sum[kPlanWaves];
  __shared__ unsigned long long pairs, steps[2];
  __shared__ int n_tiles, bad, max_chain, chunks[4];
  __shared__ int n_units[3], n_slots[3], n_comb[3];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int32_t* cu = a.cu;
  // the documents of the first batch stay in registers: every other pass starts without a trip to memory
  const int first_s = tid < a.B ? cu[tid] : 0, first_e = tid < a.B ? cu[tid + 1] : 0;
  const int cu_first = cu[0], cu_last = cu[a.B];
  auto document = [&](int b, int& s, int& e) {   // b = tid + a multiple of kPlanThreads
    s = first_s; e = first_e;
    if (b >= kPlanThreads) { s = b < a.B ? cu[b] : 0; e = b < a.B ? cu[b + 1] : 0; }
  };
  if (tid == 0) {
    bad = cu_first != 0 || cu_last != a.N;
    pairs = steps[0] = steps[1] = 0;
    n_tiles = max_chain = 0;
  }
  if (tid < 3) n_units[tid] = n_slots[tid] = n_comb[tid] = 0;
  __syncthreads();
  // ---- totals over the documents: pairs, steps of both directions, tiles, longest chains
  {
    unsigned long long my_pairs = 0, my_r = 0, my_c = 0;
    int my_bad = 0, my_tiles = 0, my_max = 0;
#pragma unroll 1
    for (int b = tid; b < a.B; b += kPlanThreads) {
      int begin, end;
      document(b, begin, end);
      const long long l = (long long)end - begin;
      if (a.B <= kSelfPlanDocs && a.N <= 0xFFFF) kept_ends(a.hdr)[b] = (uint16_t)end;   // by thread b, which may take it back
      if (l < 0) { my_bad = 1; continue; }
      my_pairs += (unsigned long long)(l * (l + 1) / 2);
      const long long T = (l + kTile - 1) / kTile, S = (l + kStep - 1) / kStep;
      my_r += (unsigned long long)(T * (T - 1) + S);
      my_c += (unsigned long long)(T * S - T * (T - 1));
      my_tiles += (int)T;
      my_max = max(my_max, (int)S);
    }
    if (my_bad) bad = 1;
    // one lane of a wave adds for all: same-address atomics of single lanes would run one by one
    if (64 * wave < a.B) {
      const int tiles = wave_total(my_tiles);
      my_max = wave_max(my_max);
      if (kOrdered) {   // at most 32768 tokens: 32 bits hold every sum
        my_pairs = (unsigned)wave_total((int)my_pairs); my_r = (unsigned)wave_total((int)my_r); my_c = (unsigned)wave_total((int)my_c);
      } else {
        my_pairs = wave_total_wide(my_pairs); my_r = wave_total_wide(my_r); my_c = wave_total_wide(my_c);
      }
      if (lane == 0 && tiles) {
        atomicAdd(&pairs, my_pairs); atomicAdd(&steps[0], my_r); atomicAdd(&steps[1], my_c);
        atomicAdd(&n_tiles, tiles);
        atomicMax(&max_chain, my_max);   // the longest row and column chains are both ceil(l / 64)
      }
    }
  }
  __syncthreads();
  varlen_attn_plan_header* hdr = a.hdr;
  if (bad || a.directions == 0) {
    if (tid < (int)(sizeof(varlen_attn_plan_header) / 4)) reinterpret_cast<int32_t*>(hdr)[tid] = 0;
    if (bad && tid < kSelfPlanDocs) kept_ends(hdr)[tid] = 0;
    __syncthreads();
    if (tid == 0) {
      const int32_t status = bad ? VARLEN_ATTN_BAD_CU_SEQLENS : VARLEN_ATTN_OK;
      hdr->status = status;
      if (a.status_copy) *a.status_copy = status;
    }
    return;
  }
  int ch[3] = {kNoSplitSteps, kNoSplitSteps, kNoSplitSteps}, line[3] = {0, 0, 0};
  int tries[3] = {0, 0, 0};
  if (!a.no_split) {
#pragma unroll
    for (int d = 0; d < 2; ++d) ch[d] = plan_chunk_steps(a.rule[d], (float)steps[d], n_tiles, a.Hq, a.force_ch[d], line[d], tries[d]);
    ch[2] = plan_dq_steps(steps, a.Hq, max(ch[0], plan_dq_shortest(steps[0], a.Hq)), a.force_ch[0]);
  }
  // Grouped-query attention: a column unit may sweep several q heads of its group (their dK, dV add up in its
  // registers: fewer and smaller group sums afterwards, none for a tile whose units sweep the whole group) as long as
  // enough units remain and the longest does not outlast the rest.
  int hpu = 1;
  if (a.g > 1) {
    if (a.force_hpu > 0 && a.g % a.force_hpu == 0) {
      hpu = a.force_hpu;
    } else if (!a.no_split) {   // unsplit plans must not depend on the rest of the microbatch
      const int whole = ch[1];
      const float col_steps = (float)steps[1], tiles = (float)n_tiles;
      const float x = col_steps * (float)a.Hq, longest_unit = a.sweep.slope * x + a.sweep.base;
      const float min_units = a.sweep.min_units + min(a.sweep.units * x, a.sweep.max_units);
#pragma unroll 1
      for (int cand = 2; cand <= a.g; ++cand) {
        if (a.g % cand) continue;
        const float shorter = (float)whole * __builtin_amdgcn_exp2f(-a.sweep.power * __builtin_amdgcn_logf((float)cand));
        const int c = a.force_ch[1] > 0 ? whole : max(kMinChunkSteps, (int)ceilf(shorter));
        // units of one head ~ steps / chunk + tiles / 2 (a cut chain rarely divides evenly)
        const float units = max(tiles, col_steps * __builtin_amdgcn_rcpf((float)c) + 0.5f * tiles) * (float)(a.Hq / cand);
        if (units >= min_units && (float)min(max_chain, c) * (float)cand <= longest_unit) { hpu = cand; ch[1] = c; }
      }
    }
  }
  const int longest = max_chain;

  // lengthen the chunks until the chunks of cut chains fit their slots; on most microbatches that one wave plans they do as they
  // are (beyond, asking costs 0.1 to 0.3 us and seldom helps)
  bool fits = kOrdered && surely_fits((float)steps[0], n_tiles, ch[0], tries[0] ? min(a.slots_cap, a.rule[0].resident) : a.slots_cap);
  if (a.directions > 1) fits = fits && surely_fits((float)steps[1], n_tiles, ch[1], a.slots_cap);   // (a dQ chunk is a row chunk or longer)
  if (!a.no_split && !fits) {
#pragma unroll 1
    for (;;) {
      if (tid < 4) chunks[tid] = 0;
      __syncthreads();
      auto count = [&](auto zero) {
        decltype(zero) all[3] = {0, 0, 0}, cut[3] = {0, 0, 0};
#pragma unroll 1
        for (int b = tid; b < a.B; b += kPlanThreads) {
          int s, e;
          document(b, s, e);
          const int T = (e - s + kTile - 1) / kTile, S = (e - s + kStep - 1) / kStep;
          count_row_chunks(T, S, ch[0], all[0], cut[0]);
          if (a.directions > 1) count_col_chunks(T, S, ch[1], all[1], cut[1]);
          if (a.directions > 2) count_row_chunks(T, S, ch[2], all[2], cut[2]);
        }
        // past the slots it is enough to know how far, up to twice as many
        auto add = [&](int i, decltype(zero) v) {
          const int sum = wave_total((int)min(v, (decltype(zero))(1 << 20)));
          if (lane == 0 && sum) atomicAdd(&chunks[i], sum);
        };
        if (64 * wave < a.B) {
#pragma unroll
          for (int d = 0; d < 3; ++d) add(d, cut[d]);
          add(3, all[0]);
        }
      };
      if (kOrdered || a.N <= (1 << 20)) count((int)0);   // no sum reaches 2^31
      else count((long long)0);
      __syncthreads();
      bool again = false;
#pragma unroll
      for (int d = 0; d < 3; ++d)
        if (next_chunk(ch[d], line[d], tries[d], (float)steps[0], chunks[d], a.slots_cap, chunks[3], a.rule[0].resident)) again = true;
      if (!again) break;
      __syncthreads();
    }
  }

  // mode 0: count the units of every cost class; mode 1: place.
  int mode = 0, shift[3] = {0, 0, 0};
#pragma unroll 1
  for (;;) {
    if (mode == 0) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        shift[d] = 0;
        while ((min(ch[d], longest) - 1) >> shift[d] >= kPlanClasses) ++shift[d];
      }
      reinterpret_cast<int*>(hist)[tid] = 0;   // 2 x 32 x waves counters: one per thread
      if (tid < kPlanThreads / 2) reinterpret_cast<int*>(hist[2])[tid] = 0;
      __syncthreads();
    }
    int row_slots_before = 0;   // cut row chains' slots so far, in tile order (single-wave form)
#pragma unroll 1
    for (int b0 = 0; b0 < a.B; b0 += kPlanThreads) {
      // ---- this batch's documents: running tile count (exclusive) by a workgroup-wide scan
      {
        int s, e;
        document(b0 + tid, s, e);
        const int T = (e - s + kTile - 1) / kTile;
        const int incl = wave_inclusive_sum(T);
        if (lane == 63) wave_sum[wave] = incl;
        doc_s[tid] = s; doc_e[tid] = e;
        __syncthreads();
        int before = 0;
#pragma unroll 1
        for (int w = 0; w < wave; ++w) before += wave_sum[w];
        doc_first_tile[tid + 1] = before + incl;
        if (tid == 0) doc_first_tile[0] = 0;
        __syncthreads();
      }
      const int batch_tiles = doc_first_tile[kPlanThreads];
      // every thread makes the same number of turns (the running sums are wave-wide scans)
#pragma unroll 1
      for (int t0 = 0; t0 < batch_tiles; t0 += kPlanThreads) {
        const int t = t0 + tid;
        const bool valid = t < batch_tiles;
        int ss = 0, ee = 0, row0 = 0, n_d[3] = {0, 0, 0}, nc_d[3] = {0, 0, 0};
        if (valid) {
          // document of tile t: the last one whose first tile is <= t (documents without tiles
          // repeat the value of their successor and are skipped by taking the last)
          int lo = 0, hi = kPlanThreads;   // doc_first_tile[lo] <= t < doc_first_tile[hi]
#pragma unroll 1
          while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (doc_first_tile[mid] <= t) lo = mid; else hi = mid;
          }
          ss = doc_s[lo]; ee = doc_e[lo];
          row0 = ss + (t - doc_first_tile[lo]) * kTile;
          n_d[0] = (min(row0 + kTile, ee) - 1 - ss) / kStep + 1;
          n_d[1] = (ee - row0 + kStep - 1) / kStep;
          nc_d[0] = (n_d[0] + ch[0] - 1) / ch[0];
          nc_d[1] = (n_d[1] + ch[1] - 1) / ch[1];
          n_d[2] = n_d[0];
          nc_d[2] = (n_d[2] + ch[2] - 1) / ch[2];
        }
        // slots of a cut row chain, numbered in tile order
        int ordered_slot0 = 0;
        if (kOrdered) {
          const int cut = nc_d[0] > 1 ? nc_d[0] : 0;
          const int incl = wave_inclusive_sum(cut);
          ordered_slot0 = row_slots_before + incl - cut;
          row_slots_before += lane_value(incl, 63);
        }
        if (valid) {
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            if (d >= a.directions) break;
            const int n = n_d[d], nc = nc_d[d], base = n / nc, rem = n % nc;
            // nc - rem chunks of `base` steps, rem chunks of base + 1 (those come first in the chain)
            int* h_lo = &hist[d][(base - 1) >> shift[d]][wave];
            int* h_hi = &hist[d][base >> shift[d]][wave];
            if (mode == 0) {
              atomicAdd(h_lo, nc - rem);
              if (rem) atomicAdd(h_hi, rem);
            } else {
              int slot0 = -1;
              if (nc > 1 || (d == 1 && a.g > hpu)) {
                if (kOrdered && d == 0) { slot0 = ordered_slot0; atomicAdd(&n_slots[0], nc); }
                else slot0 = atomicAdd(&n_slots[d], nc);
                const int ci = atomicAdd(&n_comb[d], 1);
                if (ci < a.max_combine && slot0 + nc <= a.max_slots[d])
                  a.comb[d][ci] = varlen_attn_combine_item{row0, ee, slot0, nc};
              }
              int pos_lo = atomicAdd(h_lo, nc - rem);
              int pos_hi = rem ? atomicAdd(h_hi, rem) : 0;
#pragma unroll 1
              for (int c = 0; c < nc; ++c) {
                const int first = c * base + min(c, rem), len = base + (c < rem ? 1 : 0);
                const int pos = c < rem ? pos_hi++ : pos_lo++;
                if (pos < a.max_units)
                  a.units[d][pos] = varlen_attn_unit{row0, ss, ee, first, first + len,
                                                     slot0 < 0 ? -1 : slot0 + c, len, 0};
              }
            }
          }
        }
      }
      __syncthreads();   // the batch arrays are rewritten by the next batch
    }
    if (mode == 1) break;
    // counters -> start positions: classes from the longest down, waves in order inside a class
    // (`lo`, `hi`: directions of lanes 0 .. 31 and 32 .. 63 where all classes are summed up)
    auto to_starts = [&](int d, int lo, int hi, bool active) {
      const int cls = (tid / kPlanWaves) % kPlanClasses, w = tid % kPlanWaves;
      const int own = hist[d][cls][w];
      int incl = own;   // inclusive sum over the waves of this class (adjacent lanes)
#pragma unroll
      for (int off = 1; off < kPlanWaves; off <<= 1) {
        const int o = __shfl_up(incl, off);
        if (w >= off) incl += o;
      }
      if (active && w == kPlanWaves - 1) class_total[d][cls] = incl;
      __syncthreads();
      const int total = class_total[lane < 32 ? lo : hi][kPlanClasses - 1 - (lane & 31)];   // longest class first
      int longer = wave_inclusive_sum(total);
      const int first_half = lane_value(longer, 31);
      longer -= total + (lane < 32 ? 0 : first_half);
      const int above = __shfl(longer, kPlanClasses - 1 - cls + (d == lo ? 0 : 32));
      if (active && cls == 0 && w == kPlanWaves - 1) n_units[d] = above + incl;
      if (active) hist[d][cls][w] = above + incl - own;
      __syncthreads();
    };
    to_starts(tid / (kPlanClasses * kPlanWaves), 0, 1, true);
    if (a.directions > 2) to_starts(2, 2, 2, tid < kPlanClasses * kPlanWaves);
    mode = 1;
  }
  // The capacities are worst-case bounds (tiles <= N / 128 + B; a cut chain of n > ch steps
  // takes ceil(n / ch) <= 2 n / ch chunks, and ch was lengthened until those fit), so this
  // cannot fail; if it ever does, it is an error of its own and nothing is planned.
  bool ok = true;
#pragma unroll
  for (int d = 0; d < 3; ++d) ok = ok && n_units[d] <= a.max_units && n_comb[d] <= a.max_combine && n_slots[d] <= a.max_slots[d];
  if (!ok && tid < kSelfPlanDocs) kept_ends(hdr)[tid] = 0;
  if (tid == 0) {
    hdr->status = ok ? VARLEN_ATTN_OK : VARLEN_ATTN_PLAN_OVERFLOW;
    if (a.status_copy) *a.status_copy = hdr->status;
    hdr->n_row_units = ok ? n_units[0] : 0;
    hdr->n_col_units = ok ? n_units[1] : 0;
    hdr->n_row_combine = ok ? n_comb[0] : 0;
    hdr->n_col_combine = ok ? n_comb[1] : 0;
    hdr->row_chunk_steps = ch[0];
    hdr->col_chunk_steps = ch[1];
    hdr->n_row_slots = n_slots[0];
    hdr->n_col_slots = n_slots[1];
    hdr->row_class_shift = shift[0];
    hdr->col_heads_per_unit = hpu;
    hdr->col_class_shift = shift[1];
    hdr->n_dq_units = ok ? n_units[2] : 0;
    hdr->n_dq_combine = ok ? n_comb[2] : 0;
    hdr->pairs = (int64_t)pairs;
  }
}

template <int kPlanThreads>
__global__ void __launch_bounds__(kPlanThreads) plan_kernel(PlanArgs a) {
  plan_body<kPlanThreads>(a);
}

}  // namespace

#endif  // VARLEN_ATTN_PLAN_HPP_
