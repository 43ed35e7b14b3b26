// plan.hip -- the scheduler of batches of up to kPlanPairs pairs in two
// launches, and the own keys k^ of the pass kernel.
//
// On the batches one query or a few of them make, the attention takes
// hundreds of microseconds and the general scheduler's twenty launches
// (group.hip) some 4.5 each, the longest-first order 15 to 60 more.  The
// two launches here take 7 + 5 us for 32 pairs, 10 + 17 (k^ included) for 100
// pairs of 129 tokens, 34 + 9 for 6,400 pairs, where the others took 41, 121
// and 95 to 135; a step of 32 pairs 66 -> 40 us, of 100 pairs 229 -> 174.
// One CU sorts 6,400 pairs in about 15 us, so the line is drawn where its
// LDS is full.
//   k_plan_one   block 0 holds the batch in LDS: it validates the pairs,
//                sorts them by (document, pair) with a stable radix sort,
//                finds the groups, scans their rows and items and, where the
//                units are few, puts the items in longest-first order.  The
//                other blocks write the rotary table and the norm bounds.
//   k_plan_fill  one block per sorted pair (more where the pairs are few)
//                writes its tokens' table entries, the items and work units
//                that start in it and its k^ rows; pairs without a document
//                get their zero outputs.
// The tables are those of the general scheduler, with the items themselves
// in the order of the queues (group.hip keeps an order table beside them).
#include <algorithm>

#include "attn_common.hpp"

namespace dopr {
namespace {

constexpr int kOneThreads = 1024, kOneWaves = kOneThreads / 64;
constexpr int kDigitBits = 8, kDigits = 1 << kDigitBits;
constexpr int kFillThreads = 256;

// The whole batch in the LDS of one CU: after the first loads no step of the
// plan waits for memory (with the token counts, prefix lengths and row
// offsets read from memory where they are needed, 6,400 pairs took 54 us).
constexpr int kPer = kPlanPairs / kOneThreads;  // pairs per thread
struct OneSm {
  uint32_t key[kPlanPairs];       // document id, n_docs for a skipped pair;
                                  // then each sorted pair's first row
  int32_t tok[kPlanPairs];        // stacked tokens
  int32_t len[kPlanPairs];        // prefix slots
  uint16_t order[2][kPlanPairs];  // the sort's two orders; then the first
                                  // sorted pair of each group
  uint32_t hist[kDigits * kOneWaves];  // digit-major
  uint32_t wsum[2][kOneWaves];
  int64_t row_sum;
  int32_t n_skip, n_zero, n_bad;
  float kown[2];                  // the norm bounds (full rows)
};
static_assert(sizeof(OneSm) <= 160 * 1024, "one CU's LDS");

struct OneArgs {
  Plan pl;
  PlanArgs a;
  int64_t *totals;
  int32_t *next;
  int64_t lpt_units;
  int32_t hkv, key_bits;
  // rotary table and norm bounds
  double log_theta;
  const float *inv_freq;
  const uint16_t *kw, *qw;
  int32_t D;
};

// Entries of the rotary table up to which k_plan_one's other blocks write it,
// beside the plan.  Each of them holds the LDS of the plan's block, so one runs
// per CU; a longer table is better written by a launch of its own.  Whole step,
// here -> own launch, us, at 64 entries a position: 50,000 positions 46 -> 47
// (32 pairs), 539 -> 553 (6,400); 200,000 99 -> 83, 575 -> 590; 400,000 169 ->
// 128, 646 -> 639; 1,000,000 381 -> 276, 862 -> 785.
constexpr int64_t kRopeInPlan = 16 << 20;

// Inclusive scan over the wave: row shifts, then the rows' last lanes
// broadcast into the rows behind them (DPP, no LDS round trips).
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {
#define SCAN_STEP(CTRL, ROWS)                                               \
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false)
  SCAN_STEP(0x111, 0xf);  // row_shr:1
  SCAN_STEP(0x112, 0xf);  // row_shr:2
  SCAN_STEP(0x114, 0xf);  // row_shr:4
  SCAN_STEP(0x118, 0xf);  // row_shr:8
  SCAN_STEP(0x142, 0xa);  // row_bcast:15
  SCAN_STEP(0x143, 0xc);  // row_bcast:31
#undef SCAN_STEP
  return x;
}

// Exclusive block-wide scan of one value per thread; *total gets the sum.
// Two sets of sums take turns (`set`), so one barrier orders each scan.
__device__ __forceinline__ uint32_t one_scan(OneSm &sm, int set, uint32_t v,
                                             uint32_t *total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t x = wave_scan(v);
  if (lane == 63) sm.wsum[set][wave] = x;
  __syncthreads();
  // (every wave scans the sixteen sums itself)
  const uint32_t w = wave_scan(lane < kOneWaves ? sm.wsum[set][lane] : 0);
  *total = (uint32_t)__builtin_amdgcn_readlane((int)w, kOneWaves - 1);
  const uint32_t before =
      wave ? (uint32_t)__builtin_amdgcn_readlane((int)w, wave - 1) : 0;
  return before + x - v;
}

// Validate the thread's pairs (t, t + 1024, ...) and read what the plan needs
// of them; flags and status as the general scheduler's k_pair_meta sets them.
__device__ void one_load(const OneArgs &A, OneSm &sm) {
  const PlanArgs &a = A.a;
  const int P = a.n_pairs;
  int32_t d[kPer], len[kPer];
  int32_t t0[kPer], t1[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int p = threadIdx.x + i * kOneThreads;
    const bool in = p < P;
    d[i] = in ? a.doc_ids[p] : -1;
    t0[i] = in && a.cu ? a.cu[p] : 0;
    t1[i] = in && a.cu ? a.cu[p + 1] : 1;
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i)
    len[i] = d[i] >= 0 && d[i] < a.n_docs ? a.doc_len[d[i]] : -1;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int p = threadIdx.x + i * kOneThreads;
    if (p >= P) break;
    int32_t flag = 1;
    if (a.cu) {
      if ((p == 0 && t0[i] != 0) ||
          (p == P - 1 && (int64_t)t1[i] != a.total_tokens))
        raise_status(a.status, DOPR_ERR_SEQLEN);
      if (!(t0[i] >= 0 && (int64_t)t1[i] - t0[i] >= 1 &&
            t1[i] <= a.total_tokens &&
            (int64_t)t1[i] - t0[i] <= a.max_tokens)) {
        raise_status(a.status, DOPR_ERR_SEQLEN);
        atomicAdd(&sm.n_bad, 1);
        flag = 0;
      }
    }
    if (flag && len[i] < 0) {
      raise_status(a.status, DOPR_ERR_DOC_RANGE);
      flag = 2;
      A.pl.invalid[atomicAdd(&sm.n_zero, 1)] = p;
    }
    if (flag != 1) atomicAdd(&sm.n_skip, 1);
    A.pl.pair_flag[p] = flag;
    sm.key[p] = flag == 1 ? (uint32_t)d[i] : (uint32_t)a.n_docs;
    sm.tok[p] = a.score_only ? 1 : t1[i] - t0[i];
    sm.len[p] = len[i];
  }
}

// One stable counting pass over n entries: `digit(v)` < 2^BITS of entry
// `from(e)`, placed through `put(slot, v)`.  Each wave owns a run of the
// order; lanes of one step that share a digit are ranked by the intersection
// of its bits' ballots.
template <int BITS, class From, class Digit, class Put>
__device__ __forceinline__ void one_pass(OneSm &sm, int set, int n, From from,
                                         Digit digit, Put put) {
  constexpr int N = (1 << BITS) * kOneWaves;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int run = (n + kOneThreads - 1) / kOneThreads * 64;
  const int e_end = min((wave + 1) * run, n);
  for (int i = threadIdx.x; i < N; i += kOneThreads) sm.hist[i] = 0;
  __syncthreads();
  for (int e = wave * run + lane; e < e_end; e += 64)
    atomicAdd(&sm.hist[digit(from(e)) * kOneWaves + wave], 1u);
  __syncthreads();
  {
    constexpr int PER = N / kOneThreads;
    uint32_t c[PER], sum = 0, tot;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      c[i] = sm.hist[threadIdx.x * PER + i];
      sum += c[i];
    }
    uint32_t at = one_scan(sm, set, sum, &tot);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      sm.hist[threadIdx.x * PER + i] = at;
      at += c[i];
    }
  }
  __syncthreads();
  // (a wave's cursors: read by every lane, then moved by the first lane of
  // each digit; LDS operations of a wave run in order)
  volatile uint32_t *cursor = sm.hist;
  const uint64_t below = (1ull << lane) - 1;
  for (int e0 = wave * run; e0 < e_end; e0 += 64) {
    const bool in = e0 + lane < e_end;
    const uint32_t v = in ? from(e0 + lane) : 0;
    const uint32_t d = in ? digit(v) : 0;
    uint64_t same = __ballot(in);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
      const uint64_t m = __ballot((d >> b) & 1);
      same &= (d >> b) & 1 ? m : ~m;
    }
    if (in) {
      const uint32_t base = cursor[d * kOneWaves + wave];
      const int rank = __popcll(same & below);
      put(base + rank, v);
      if (rank == 0)
        cursor[d * kOneWaves + wave] = base + (uint32_t)__popcll(same);
    }
  }
  __syncthreads();
}

// Sort of the pairs by (key, pair index), 8 bits a pass; returns the order's
// buffer.
__device__ int one_sort(const OneArgs &A, OneSm &sm) {
  int cur = 0;
  for (int shift = 0; shift < A.key_bits || shift == 0;
       shift += kDigitBits) {
    const uint16_t *prev = sm.order[cur];
    uint16_t *to = sm.order[cur ^ 1];
    one_pass<kDigitBits>(
        sm, cur, A.a.n_pairs,
        [&](int e) { return shift ? (uint32_t)prev[e] : (uint32_t)e; },
        [&](uint32_t v) { return (sm.key[v] >> shift) & (kDigits - 1); },
        [&](uint32_t at, uint32_t v) { to[at] = (uint16_t)v; });
    cur ^= 1;
  }
  return cur;
}

__global__ __launch_bounds__(kOneThreads) void k_plan_one(OneArgs A) {
  __shared__ OneSm sm;
  const Plan &pl = A.pl;
  const PlanArgs &a = A.a;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if (blockIdx.x == 1) {
    norm_bound(A.kw, A.qw, A.D, reinterpret_cast<float *>(sm.hist), pl.kown,
               pl.unit_w);
    return;
  }
  if (blockIdx.x > 1) {
    rope_entry(pl.rope, pl.rope_pos, A.D / 2, A.log_theta, A.inv_freq,
               (int64_t)(blockIdx.x - 2) * kOneThreads + t);
    return;
  }
  if (t == 0) sm.n_skip = sm.n_zero = sm.n_bad = 0;
  if (t < kCounters) pl.counters[t] = 0;
  if (t < kNextQueues) A.next[t] = 0;
  if (t < 64) reinterpret_cast<int32_t *>(pl.zero)[t] = 0;
  __syncthreads();
  const int P = a.n_pairs;
  // (the pass kernel's items follow from the norm bounds: formed here too)
  if (a.exact_items) {  // block-uniform
    norm_bound(A.kw, A.qw, A.D, reinterpret_cast<float *>(sm.hist), sm.kown,
               pl.unit_w);
    __syncthreads();
  }
  const int32_t rows_per_item = plan_cut(a, sm.kown).rows_per_item;
  one_load(A, sm);
  __syncthreads();
  const int n_valid = P - sm.n_skip;
  const int cur = one_sort(A, sm);
  const uint16_t *order = sm.order[cur];
  uint16_t *first = sm.order[cur ^ 1];  // first sorted pair of each group

  // groups and rows: each thread takes consecutive sorted pairs
  const int per = (n_valid + kOneThreads - 1) / kOneThreads;
  const int s0 = t * per, s1 = min(s0 + per, n_valid);
  uint32_t rows = 0;
  uint32_t head = 0;  // bit i: pair s0 + i starts a group
  uint32_t doc[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int s = s0 + i;
    if (s >= s1) break;
    const int p = order[s];
    doc[i] = sm.key[p];
    if (s == 0 || doc[i] != sm.key[order[s - 1]]) head |= 1u << i;
    rows += (uint32_t)sm.tok[p] * (uint32_t)a.n_rep;
  }
  uint32_t n_groups, n_rows, n_items = 0;
  uint32_t g = one_scan(sm, 0, __popc(head), &n_groups);
  uint32_t r = one_scan(sm, 1, rows, &n_rows);
  // Token ranges that follow one another stack at most the rows the plan
  // holds (below 2^31).  With a malformed range among them they may overlap
  // and stack more: the batch is then not run.
  bool fits = true;
  if (sm.n_bad > 0) {  // block-uniform
    if (t == 0) sm.row_sum = 0;
    __syncthreads();
    for (int s = t; s < n_valid; s += kOneThreads)
      atomicAdd(reinterpret_cast<unsigned long long *>(&sm.row_sum),
                (unsigned long long)sm.tok[order[s]] *
                    (unsigned long long)a.n_rep);
    __syncthreads();
    fits = sm.row_sum <= a.rows_cap;
  }
  // (the scans' barriers: every thread has read its keys)
  uint32_t *row_of = sm.key;
  if (fits) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int s = s0 + i;
      if (s >= s1) break;
      const int p = order[s];
      if (head >> i & 1) {
        pl.group_doc[g] = (int32_t)doc[i];
        pl.group_ptr[g] = s;
        first[g] = (uint16_t)s;
        ++g;
      }
      row_of[s] = (uint32_t)r;
      pl.pair_order[s] = p;
      pl.prow[s] = r;
      pl.tmp_order[s] = (int32_t)g - 1;  // the pair's group
      r += (int64_t)sm.tok[p] * a.n_rep;
    }
    if (t == 0) {
      pl.group_ptr[n_groups] = n_valid;
      pl.prow[n_valid] = n_rows;
      pl.spair[n_valid] = make_int4(0, 0, (int32_t)n_rows, 0);
    }
  }
  __syncthreads();

  // items per group, scanned: in group order, or longest first (costliest
  // class first, group order within a class) while the CUs get few units
  const int G = fits ? (int)n_groups : 0;
  const int gper = (G + kOneThreads - 1) / kOneThreads;
  const int g0 = t * gper, g1 = min(g0 + gper, G);
  auto group_rows = [&](int i) {
    return (i + 1 < G ? row_of[first[i + 1]] : n_rows) - row_of[first[i]];
  };
  auto group_items = [&](int i) {
    return (group_rows(i) + (uint32_t)rows_per_item - 1) /
           (uint32_t)rows_per_item;
  };
  uint32_t items = 0;
  for (int i = g0; i < g1; ++i) items += group_items(i);
  uint32_t at = one_scan(sm, 0, items, &n_items);
  const bool enough = (int64_t)n_items <= pl.items_cap;
  if ((int64_t)n_items * A.hkv > A.lpt_units) {
    for (int i = g0; i < g1; ++i) {
      pl.item_scan[i] = at;
      at += group_items(i);
    }
  } else {
    // the groups by class, stable, then their items scanned in that order
    // (the sorted groups take the token counts' place, read for the last
    // time above)
    uint16_t *sorted = reinterpret_cast<uint16_t *>(sm.tok);
    static_assert(kCostBuckets <= 64, "six bits a class");
    one_pass<6>(
        sm, 1, G, [&](int e) { return (uint32_t)e; },
        [&](uint32_t v) {
          return (uint32_t)cost_class(group_rows(v), sm.len[order[first[v]]]);
        },
        [&](uint32_t slot, uint32_t v) { sorted[slot] = (uint16_t)v; });
    items = 0;
    for (int i = g0; i < g1; ++i) items += group_items(sorted[i]);
    uint32_t tot;
    at = one_scan(sm, 0, items, &tot);
    for (int i = g0; i < g1; ++i) {
      pl.item_scan[sorted[i]] = at;
      at += group_items(sorted[i]);
    }
  }
  const bool ok = fits && enough;
  if (!ok)
    for (int p = t; p < P; p += kOneThreads)
      if (pl.pair_flag[p] == 1) pl.pair_flag[p] = 0;
  if (t == 0) {
    if (!ok) raise_status(a.status, DOPR_ERR_SEQLEN);
    A.totals[kTotDocs] = ok ? (int64_t)n_groups << 32 | n_valid : 0;
    A.totals[kTotRows] = ok ? n_rows : 0;
    A.totals[kTotItems] = ok ? n_items : 0;
    A.totals[kTotUnits] = 0;  // (the items are in the queues' order)
    pl.counters[kCntInvalid] = sm.n_zero;
    if (ok && a.exact_items && all_over(a.c, sm.kown))
      pl.counters[kCntFix] = (int32_t)n_items * A.hkv;  // (k_plan_fill lists)
  }
}

// ---------------------------------------------------------------------------
// k^ of one pair's keys: RMSNorm, gain and rotation of every online key at
// positions L + j, for every kv head, with the arithmetic of the block
// kernels' own-key staging (own_stage), rounded to bf16 and written as
// k^ [Hkv][Ntok][D].  The pass kernel then copies own keys like prefix keys,
// and a pair's keys are normed once per batch instead of once per pass that
// reads them.  Block `part` of `parts` takes every parts-th step of rows.
// Bound by memory: 2 x 1.7 GB in 0.66 ms (5.1 TB/s) at 825,600 tokens of 8
// kv heads.
constexpr int kKhatRowsPerStep = 2;

template <int D>
__device__ __forceinline__ void khat_pair(const KhatParams &P, int4 sp, int L,
                                          int part, int parts) {
  constexpr int NSUB = D / 16, ROWS = kFillThreads / NSUB;
  const int tok0 = sp.x, T = sp.y;
  const int t = threadIdx.x;
  const int sub = t % NSUB;
  const uint4 g0 = *reinterpret_cast<const uint4 *>(P.kw + 8 * sub);
  const uint4 g1 = *reinterpret_cast<const uint4 *>(P.kw + D / 2 + 8 * sub);
  const int64_t n_rows = (int64_t)T * P.Hkv;
  // KB rows per thread and step, every row's loads issued before the first
  // is used (the stores of one step cannot be moved above the next step's
  // loads by the compiler, so one row per step leaves one load in flight)
  constexpr int KB = kKhatRowsPerStep;
  for (int64_t r0 = (int64_t)part * KB * ROWS + t / NSUB; r0 < n_rows;
       r0 += (int64_t)parts * KB * ROWS) {
    uint4 a0[KB], a1[KB];
    const float4 *cq[KB];
    int j[KB], g[KB];
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      const int64_t rr = r0 + k * ROWS < n_rows ? r0 + k * ROWS : r0;
      j[k] = (int)(rr / P.Hkv);
      g[k] = (int)(rr % P.Hkv);
      const uint16_t *kr = P.k + ((int64_t)(tok0 + j[k]) * P.Hkv + g[k]) * D;
      a0[k] = *reinterpret_cast<const uint4 *>(kr + 8 * sub);
      a1[k] = *reinterpret_cast<const uint4 *>(kr + D / 2 + 8 * sub);
      cq[k] = reinterpret_cast<const float4 *>(
          P.rope + (int64_t)(L + j[k]) * (D / 2) + 8 * sub);
    }
    float4 c[KB][4];
#pragma unroll
    for (int k = 0; k < KB; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i) c[k][i] = cq[k][i];
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      if (k > 0 && r0 + k * ROWS >= n_rows) break;
      float x[16];
      khat_part<D>(a0[k], a1[k], g0, g1, c[k][0], c[k][1], c[k][2], c[k][3],
                   true, P.eps, P.norm != 0, x);
      uint16_t *o = P.kh + ((int64_t)g[k] * P.ntok + tok0 + j[k]) * D;
      *reinterpret_cast<uint4 *>(o + 8 * sub) = as_uint4(to_bf16x8(x));
      *reinterpret_cast<uint4 *>(o + D / 2 + 8 * sub) =
          as_uint4(to_bf16x8(x + 8));
    }
  }
}

// The same for every sorted pair of a batch the general scheduler planned,
// one block per pair; for none where the pass kernel has nothing to do.
template <int D>
__global__ __launch_bounds__(kFillThreads) void k_own_khat(KhatParams P) {
  const int s = blockIdx.x;
  if (s >= plan_pairs(P.totals, P.rows_cap) || all_over(P.c, P.kown)) return;
  khat_pair<D>(P, P.spair[s], P.doc_len[P.doc_ids[P.pair_order[s]]], 0, 1);
}

struct FillArgs {
  Plan pl;
  PlanArgs a;
  StoreView sv;
  KhatParams k;      // k.kh NULL: no pass kernel
  UnitArgs u;
  uint16_t *out;     // outputs of the pairs without a document
  float *lse;
  int32_t hq, parts;
};

// The items whose first row lies in sorted pair s (its record sp), with
// their work units: the pair is then the item's first one, and a document
// with hundreds of items is spread over its pairs' blocks.
__device__ __forceinline__ void pair_items(const FillArgs &A, const int4 &sp,
                                           int s) {
  const Plan &pl = A.pl;
  const PlanArgs a = plan_cut(A.a, A.pl.kown);
  const bool over = A.k.kh && all_over(a.c, pl.kown);
  const int g = pl.tmp_order[s];
  const int64_t base = pl.prow[pl.group_ptr[g]];
  const int64_t R = pl.prow[pl.group_ptr[g + 1]] - base;
  const int64_t n_it = (R + a.rows_per_item - 1) / a.rows_per_item;
  const int64_t at = pl.item_scan[g];
  const int64_t z = sp.z, end = pl.prow[s + 1];
  // the first item that starts at or behind the pair's first row
  int64_t lo = a.exact_items ? (z - base + a.rows_per_item - 1) /
                                   a.rows_per_item
                             : (z - base) * n_it / R;
  while (lo > 0 && item_start(a, base, R, n_it, lo - 1) >= z) --lo;
  while (lo < n_it && item_start(a, base, R, n_it, lo) < z) ++lo;
  const int hkv = A.k.kh ? A.sv.n_kv_heads : 1;
  for (int64_t i = threadIdx.x;; i += kFillThreads) {
    const int64_t it = lo + i / hkv;
    if (it >= n_it) break;
    const int64_t b0 = item_start(a, base, R, n_it, it);
    if (b0 >= end) break;
    const int h = (int)(i % hkv);
    const int4 item = make_int4(
        g, (int32_t)b0, (int32_t)item_start(a, base, R, n_it, it + 1), s);
    if (h == 0) pl.items[at + it] = item;
    if (over)
      pl.fix[(at + it) * hkv + h] = (int32_t)((at + it) * hkv + h) |
                                    kFixUnscored;
    else if (A.k.kh)
      write_unit(pl, A.sv, A.u, (at + it) * hkv + h, item, sp, h);
  }
}

template <int D>
__global__ __launch_bounds__(kFillThreads) void k_plan_fill(FillArgs A) {
  const Plan &pl = A.pl;
  const PlanArgs &a = A.a;
  const int64_t *totals = A.k.totals;
  const int n_valid = (int)(totals[kTotDocs] & 0xffffffff);
  const int s = blockIdx.x / A.parts, part = blockIdx.x % A.parts;
  if (s >= n_valid) {
    const int i = s - n_valid;
    if (part == 0 && i < pl.counters[kCntInvalid])
      zero_pair(pl.invalid[i], a.score_only ? nullptr : a.cu, A.hq, D,
                A.out, A.lse);
    return;
  }
  const int p = pl.pair_order[s];
  const int tok0 = a.cu[p];
  const int4 sp = make_int4(tok0, a.cu[p + 1] - tok0, (int32_t)pl.prow[s], 0);
  if (part == 0) {
    if (threadIdx.x == 0) pl.spair[s] = sp;
    const int stacked = a.score_only ? 1 : sp.y;
    const int64_t u0 = sp.z / a.n_rep;
    for (int j = threadIdx.x; j < stacked; j += kFillThreads)
      pl.utok[u0 + j] = make_int2(sp.x + (sp.y - 1 - j), sp.y - 1 - j);
    // owners of the 32-row blocks that start in this pair
    const int64_t end = (int64_t)sp.z + (int64_t)stacked * a.n_rep;
    const int64_t b1 = std::min<int64_t>((end + 31) >> 5, pl.blk_cap);
    for (int64_t b = (((int64_t)sp.z + 31) >> 5) + threadIdx.x; b < b1;
         b += kFillThreads)
      pl.blk_pair[b] = s;
  }
  if (part == 0) pair_items(A, sp, s);
  if (A.k.kh && !all_over(a.c, pl.kown))
    khat_pair<D>(A.k, sp, a.doc_len[a.doc_ids[p]], part, A.parts);
}

template <int D>
hipError_t launch_fill(const FillArgs &f, hipStream_t s) {
  hipLaunchKernelGGL(k_plan_fill<D>, dim3(f.a.n_pairs * f.parts),
                     dim3(kFillThreads), 0, s, f);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_khat(int D, const KhatParams &kp, int32_t n_pairs,
                       hipStream_t s) {
  if (n_pairs == 0) return hipSuccess;
  if (D == 128)
    hipLaunchKernelGGL(k_own_khat<128>, dim3((unsigned)n_pairs),
                       dim3(kFillThreads), 0, s, kp);
  else
    hipLaunchKernelGGL(k_own_khat<64>, dim3((unsigned)n_pairs),
                       dim3(kFillThreads), 0, s, kp);
  return hipGetLastError();
}

hipError_t launch_plan_one(const AttnCall &c, const Plan &pl,
                           const PlanShape &shape, const PlanArgs &pa,
                           int64_t lpt_units, hipStream_t s) {
  const dopr_attn_args_t *a = c.a;
  OneArgs o{};
  o.pl = pl;
  o.a = pa;
  o.totals = plan_totals(pl);
  o.next = plan_next(pl);
  o.lpt_units = lpt_units;
  o.hkv = c.st->n_kv_heads;
  o.key_bits = 0;
  while (o.key_bits < 31 && (c.st->n_docs >> o.key_bits) > 0) ++o.key_bits;
  o.log_theta = std::log((double)a->rope_theta);
  o.inv_freq = a->rope_inv_freq;
  o.kw = static_cast<const uint16_t *>(a->k_norm_w);
  o.qw = static_cast<const uint16_t *>(a->q_norm_w);
  o.D = c.st->head_dim;
  const int64_t entries = (int64_t)pl.rope_pos * (o.D / 2);
  unsigned rope = (unsigned)((entries + kOneThreads - 1) / kOneThreads);
  if (entries > kRopeInPlan) {
    const hipError_t e = launch_rope_table(c, pl, s);
    if (e != hipSuccess) return e;
    rope = 0;
  }
  hipLaunchKernelGGL(k_plan_one, dim3(2 + rope), dim3(kOneThreads), 0, s, o);
  return hipGetLastError();
}

hipError_t launch_plan_fill(const AttnCall &c, const Plan &pl,
                            const PlanShape &shape, const PlanArgs &pa,
                            hipStream_t s) {
  const dopr_attn_args_t *a = c.a;
  FillArgs f{};
  f.pl = pl;
  f.a = pa;
  f.sv = c.st->view();
  f.k = khat_params(c, pl);
  f.u = unit_args(c);
  f.out = static_cast<uint16_t *>(a->out);
  f.lse = a->lse;
  f.hq = a->n_q_heads;
  // blocks per pair: enough for a few thousand in all, each with at least
  // one step of rows
  f.parts = 1;
  if (pl.kh) {
    const int64_t steps = ((int64_t)a->max_tokens * c.st->n_kv_heads *
                               c.st->head_dim / 16 +
                           kKhatRowsPerStep * kFillThreads - 1) /
                          (kKhatRowsPerStep * kFillThreads);
    f.parts = (int32_t)std::max<int64_t>(
        1, std::min<int64_t>(steps, 2048 / a->n_pairs));
  }
  return c.st->head_dim == 128 ? launch_fill<128>(f, s) : launch_fill<64>(f, s);
}

}  // namespace dopr
