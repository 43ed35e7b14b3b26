// internal.hpp -- shared declarations of the DoPR HIP library (not part of
// the public ABI; the public contract is include/dopr.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>
#include <cstdint>

#include "dopr.h"

namespace dopr {

// Head sizes: 128 (Qwen3, Llama 3) and 64 (Llama 3.2 1B).  Everything sized
// for the largest uses kHeadDim; per-call code takes the store's head_dim.
constexpr int kHeadDim = 128;
constexpr int kAlign = 256;
// Longest prefix for which last-layer scoring runs one wave per 32-row work
// unit (the kernel variant and the planner's item size both follow it).
constexpr int32_t kScoreRowsMaxLen = 512;

// The attention's reference-free softmax serves a work unit when every
// logit (log2 units) lies in [-kNoRefBound, kNoRefBound].
constexpr float kNoRefBound = 64.f;

// Largest attention plan dopr_prefix_attn_noalloc lays out in the library's
// own scratch array (one copy per device).
constexpr size_t kNoAllocScratchBytes = DOPR_NOALLOC_SCRATCH_BYTES;

// Stacked rows of a work unit of the pass kernel: a 32-row tile for each of
// a block's four waves.
constexpr int32_t kPassRows = 128;

// The automatic choice of a full layer: the pass kernel, except at head size
// 64 for batches of at most kPassRows stacked rows with a prefix of more than
// kOneTileSlots slots.  There a handful of units wait for their prefixes alone,
// and a block kernel of eight waves has 512 slots of them on their way at
// once: block kernel -> pass kernel, us per call, 1 to 104 rows 29.3 to 33.2 ->
// 31.1 to 34.6 (500 slots), 40.2 to 49.4 -> 44.7 to 51.6 (1,500); 192 to 252
// rows 36.2 -> 35.0 and 49.0 -> 48.3.  Elsewhere, 1 to 32 kv heads, 1 to 8 q
// heads per kv head, 1 to 129 tokens, 8 to 1,500 slots, the pass kernel is the
// faster one or within 5 %: head size 128, 1 to 400 rows 57 -> 54, 486 -> 330
// (1,500 slots, one or 400 documents); 4,128 rows 87 -> 38 (head size 64, 500
// slots); 12,000 rows 2,650 -> 1,596 (1,500 slots), 360 -> 301 (8 slots);
// 250,000 rows 1,290 -> 1,096, 2,000 -> 1,890.  The worst of 800 batches: 82.5
// -> 86.9 (3,500 pairs of one token on 8 slots, 2 kv heads).
constexpr int32_t kOneTileSlots = 256;

// Rows per work item of the block kernels, which walk an item in passes, unless
// the caller sets them.
constexpr int32_t kBlockRows = 2048;

// Fix-up list entries: work unit index, plus this bit when the unit was not
// computed by the fast pass (its logit bound exceeds kNoRefBound); those
// run the bounded-reference mode first, the others the exact mode.
constexpr int32_t kFixUnscored = 1 << 30;

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
__host__ __device__ inline int32_t pad8(int32_t n) { return (n + 7) & ~7; }

// Device status words at the head of every store pool.
enum StatusSlot { kStatusFirstError = 0, kStatusWords = 64 };

// Store layout inside the caller's pool:
//   [status words | doc_len int32[n_docs] | doc_off int64[n_docs] |
//    kmax fp32[n_docs][n_layers][Hkv] | payload]
// kmax holds an upper bound on the L2 norm of every stored key of a
// document's (layer, kv head) slice (0 when L = 0); the attention kernel uses
// it to bound logits.
// Each resident document owns one contiguous block of the payload; for layer
// l and kv head g the block holds
//   K  [L][D]   at  blk + l*Hkv*D*(L+Lp) + g*L*D
//   Vt [D][Lp]  at  blk + l*Hkv*D*(L+Lp) + Hkv*L*D + g*D*Lp
// with Lp = L rounded up to 8 (V is stored transposed so the PV contraction
// over keys reads 16-byte runs; the pad columns are zero).
struct StoreView {
  const int32_t *doc_len;  // [n_docs], -1 = not resident
  const int64_t *doc_off;  // [n_docs], element offset of the doc block
  float *kmax;             // [n_docs][n_layers][Hkv] key-norm bound
  uint16_t *payload;
  int64_t n_docs;
  int32_t n_layers, n_kv_heads, head_dim;
};

__host__ __device__ inline int64_t layer_block_elems(int32_t L, int32_t hkv,
                                                     int32_t D) {
  return (int64_t)hkv * D * ((int64_t)L + pad8(L));
}
__host__ __device__ inline int64_t k_offset(int64_t blk, int32_t L, int32_t hkv,
                                            int32_t layer, int32_t g,
                                            int32_t D) {
  return blk + layer * layer_block_elems(L, hkv, D) + (int64_t)g * L * D;
}
__host__ __device__ inline int64_t vt_offset(int64_t blk, int32_t L,
                                             int32_t hkv, int32_t layer,
                                             int32_t g, int32_t D) {
  return blk + layer * layer_block_elems(L, hkv, D) + (int64_t)hkv * L * D +
         (int64_t)g * D * pad8(L);
}

}  // namespace dopr

struct dopr_store {
  int32_t n_layers, n_kv_heads, head_dim;
  int64_t n_docs;
  char *pool;
  size_t pool_bytes;
  int32_t *d_status;
  int32_t *d_len;
  int64_t *d_off;
  float *d_kmax;
  uint16_t *d_payload;
  int32_t max_len;  // largest L over resident documents
  int device;
  dopr::StoreView view() const {
    return {d_len, d_off, d_kmax, d_payload, n_docs, n_layers, n_kv_heads,
            head_dim};
  }
};

namespace dopr {

// ---------------------------------------------------------------------------
// Groups with more pairs than this are put in pair order by a sort (one
// block per group) instead of a scan of the group per pair.
constexpr int32_t kBigGroup = 256;
// Cost classes of work units for the longest-first order: floor(log2) of
// stacked rows x (prefix slots + 32).
constexpr int32_t kCostBuckets = 40;

// The plan's int64 totals.
enum Total {
  kTotDocs = 0,   // (distinct docs << 32) | valid pairs
  kTotRows = 1,   // stacked rows of the valid pairs
  kTotItems = 2,  // work items
  kTotUnits = 3,  // 1 if the queues follow the longest-first order, else 0
  kTotals = 4
};

// Work unit handed out as the `slot`-th claim of queue `queue` (0..7):
// queue q serves the units w with w % 8 == q, in natural order (w = q +
// 8 * slot) when qorder is null, else costliest class first as the
// planner's qorder lists them; n_work when the queue is empty.
__device__ __forceinline__ int64_t unit_at(const int32_t *qorder, int queue,
                                           int64_t slot, int64_t n_work) {
  if (!qorder) {
    const int64_t w = queue + 8 * slot;
    return w < n_work ? w : n_work;
  }
  const int64_t per = n_work / 8, rem = n_work % 8;
  const int64_t n_q = per + (queue < rem ? 1 : 0);
  if (slot >= n_q) return n_work;
  const int64_t start = queue * per + (queue < rem ? queue : rem);
  return qorder[start + slot];
}

// The same in 32 bits: argument validation keeps every unit number (and
// n_work) below 2^31.
__device__ __forceinline__ int unit_at32(const int32_t *qorder, int queue,
                                         int slot, int n_work) {
  if (!qorder) {
    // slot >= the queue's unit count, tested without forming q + 8 * slot
    if (slot >= (n_work - queue + 7) / 8) return n_work;
    return queue + 8 * slot;
  }
  const int per = n_work / 8, rem = n_work % 8;
  const int n_q = per + (queue < rem ? 1 : 0);
  if (slot >= n_q) return n_work;
  const int start = queue * per + (queue < rem ? queue : rem);
  return qorder[start + slot];
}

// A work unit of the pass kernel (one item for one kv head), 64 bytes.
// Addresses are (low, high) words.
struct PassUnit {
  int32_t u0;        // stacked token of its first row
  int32_t rows;      // rows (at most 128) | first row's head in the group << 8
  int32_t s;         // first sorted pair; sign bit: over the logit bound
  int32_t L;         // prefix slots
  int32_t k[2];      // the document's K slice (this layer and head)
  int32_t vt[2];     // its V^T slice
  int32_t own_k[2];  // k^ of the first pair's first token (this head)
  int32_t own_v[2];  // its v
  int32_t tok0, T;   // the first pair's first token and token count
  int32_t jmax;      // its latest position in the unit
  int32_t g;         // kv head
};
static_assert(sizeof(PassUnit) == 64, "one 16-word scalar load");

enum NextSlots { kNextQueues = 16 };  // 8 XCD queues + the SAFE pass

// Per-call plan built on the device by the grouping kernels (workspace).
enum Counter {
  kCntValid = 0,     // pairs with a valid, resident document
  kCntGroups = 1,    // distinct documents among them
  kCntItems = 2,     // attention work items
  kCntInvalid = 3,   // pairs whose outputs must be zeroed
  kCntRows = 4,      // stacked rows (tokens * n_rep) of valid pairs (low)
  kCntFix = 5,       // work units queued for the exact (SAFE) pass
  kCntBig = 6,       // groups of more than kBigGroup pairs (ordered apart)
  kCounters = 16
};

struct Plan {
  int32_t *counters;    // [kCounters]
  int32_t *cnt;         // [n_docs]   pairs per document
  int32_t *fill;        // [n_docs]   placement cursor per document
  int64_t *doc_scan;    // [n_docs]   (has_pairs << 32 | count), scanned
  int64_t *blk;         // scan block sums
  int32_t *pair_flag;   // [P] 1 = valid, 0 = skip, 2 = zero outputs
  int32_t *invalid;     // [P] pairs whose outputs are zeroed
  int32_t *tmp_order;   // [P] (plan.hip: the sorted pairs' groups)
  int32_t *pair_order;  // [P]
  int4 *big;            // [P / (kBigGroup + 1) + 1] groups of more than
                        // kBigGroup pairs: (first slot, pairs, doc, group)
  int32_t *qorder;      // [items_cap * Hkv] work units by queue (w % 8),
                        // costliest class first within each queue, unit
                        // order within a class (when totals[kTotUnits]
                        // is 1)
  uint8_t *item_cls;    // [items_cap] cost class of each item's group
  int32_t *group_doc;   // [P]
  int32_t *group_ptr;   // [P+1]
  int64_t *prow;        // [P+1] stacked-row offsets, sorted pair order
  int64_t *item_scan;   // [P+1] work items per group, scanned
  int32_t *blk_pair;    // [blk_cap] sorted pair owning row 32*b
  int4 *items;          // [items_cap] (group, row0, row1, first sorted pair)
  int32_t *fix;         // [items_cap * Hkv] work units for the SAFE pass
  int4 *spair;          // [P+1] sorted pair: (tok0, T, first stacked row)
  int2 *utok;           // [stacked tokens] (batch token, position)
  float *part;          // [P][Hq][3] score-head partial sums (score mode)
  float *kown;          // [2] bounds on |k^| (own keys) and |q^|: sqrt(D) max|w|
                        // (0 when there is no QK-norm: no bound is known)
  uint16_t *unit_w;     // [D] bf16 ones: the gains when there is no QK-norm
  float2 *rope;         // [rope_pos][D/2] (cos, sin)
  uint16_t *kh;         // [Hkv][Ntok][D] own keys k^ (pass kernel), or NULL
  PassUnit *units;      // [items_cap * Hkv] work units (pass kernel)
  uint16_t *zero;       // 256 zero bytes (the pass kernel loads them past row ends)
  int32_t items_cap;
  int32_t blk_cap;
  int32_t rope_pos;
  int64_t scan_blocks_cap;
};

// Scheduler arguments of one call.
struct PlanArgs {
  const int32_t *doc_ids, *cu, *doc_len;
  int64_t n_docs, total_tokens;
  int32_t n_pairs, n_rep, max_tokens, rows_per_item;
  int32_t *status;
  bool score_only;
  bool exact_items;
  int64_t rows_cap;  // stacked rows the plan's tables hold
  int32_t rows_over;  // rows per item where every unit is over the bound
  float c;            // softmax_scale * log2(e)
};

// Groups and valid pairs of a batch, from its totals.  Token ranges that
// follow one another stack at most rows_cap rows; with a malformed range among
// them they may overlap and stack more, and such a batch is not run: none.
__device__ inline int32_t plan_groups(const int64_t *totals, int64_t rows_cap) {
  return totals[kTotRows] > rows_cap ? 0 : (int32_t)(totals[kTotDocs] >> 32);
}
__device__ inline int32_t plan_pairs(const int64_t *totals, int64_t rows_cap) {
  return totals[kTotRows] > rows_cap
             ? 0 : (int32_t)(totals[kTotDocs] & 0xffffffff);
}

// Whether the gains alone put every unit of a call over the logit bound: the
// bound of a unit's keys is at least that of its own keys, kown[0].  The pass
// kernel then has nothing to do: the plan cuts the rows into items for the
// exact pass, which walks an item with a prefix staged once for all of its
// rows, lists every unit for it (plan_cut) and leaves k^ out (6,400 pairs of 129
// tokens on 256 slots, 32 q / 8 kv heads: 13780 -> 13110 us).
__device__ inline bool all_over(float c, const float *kown) {
  return c * kown[1] * kown[0] * 1.001f > kNoRefBound;
}
// Rows of those items (rows: stacked rows times kv heads): the block kernels'
// size in a large batch, less where the CUs would not get kOverUnitsPerCu units
// each, down to one pass of the exact kernel.  Gains five times the usual, us
// per call (k^ formed) with items of 128, 512 and 2,048 rows: 6,400 pairs of 129 tokens on
// 256 slots (32 q / 8 kv heads) 18230, 14840, 13780; 1,600 of 65 on 50 documents
// of 512 slots 2700, 2650, 2750; 100 of 129 on 256 slots 320, 280, 290.  Six
// times, where many a row takes the exact mode and its unit with it: 30,000 rows
// of 27 documents of 1,500 slots, one kv head, 170 (2,048 rows: 1,460);
// 59 pairs of 129 tokens on one document, 2 kv heads, 92 (460).
constexpr int32_t kOverUnitsPerCu = 8;
inline int32_t over_rows(int64_t rows, int n_cu) {
  const int64_t per = rows / ((int64_t)kOverUnitsPerCu * n_cu) / kPassRows;
  return per < 1 ? kPassRows
         : per >= kBlockRows / kPassRows ? kBlockRows
                                         : (int32_t)per * kPassRows;
}
__device__ inline PlanArgs plan_cut(PlanArgs a, const float *kown) {
  if (a.exact_items && all_over(a.c, kown)) {
    a.rows_per_item = a.rows_over;
    a.exact_items = false;
  }
  return a;
}

// The longest-first cost class of a document group: kCostBuckets - 1 -
// floor(log2(stacked rows * (prefix slots + 32))), clamped to the buckets
// (0 = costliest).
__device__ inline uint8_t cost_class(int64_t rows, int32_t L) {
  const int64_t cost = rows * ((int64_t)L + 32);
  const int b = cost > 0 ? 63 - __clzll((unsigned long long)cost) : 0;
  return (uint8_t)(kCostBuckets - 1 - (b < kCostBuckets ? b : kCostBuckets - 1));
}

// Bounds on the norms of every own key k^ and every query q^, each of the
// form RoPE(RMSNorm(x) * w): an RMS-normed vector has norm <= sqrt(D), the
// gain scales it by at most max|w|, rotation keeps it, and bf16 rounding
// adds at most 2^-8.  bound[0] is for keys (w_k), bound[1] for queries.
// Without QK-norm (no gains) no bound is known: both are written as 0 and
// unit_w gets the unit gains the attention kernel multiplies by.  One
// thread per head dim (64 or 128; a block's further threads only meet the
// barrier); red: four floats of LDS.
__device__ inline void norm_bound(const uint16_t *kw, const uint16_t *qw,
                                  int D, float *red, float *bound,
                                  uint16_t *unit_w) {
  const int t = threadIdx.x;
  float a = 0.f, b = 0.f;
  if (t < D) {
    if (!kw) unit_w[t] = 0x3F80;  // bf16 1.0
    if (kw) a = fabsf(__uint_as_float((uint32_t)kw[t] << 16));
    if (qw) b = fabsf(__uint_as_float((uint32_t)qw[t] << 16));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      a = fmaxf(a, __shfl_xor(a, off, 64));
      b = fmaxf(b, __shfl_xor(b, off, 64));
    }
    if ((t & 63) == 0) {
      red[t >> 6] = a;
      red[2 + (t >> 6)] = b;
    }
  }
  __syncthreads();
  if (t < 2) {
    const float m = D > 64 ? fmaxf(red[2 * t], red[2 * t + 1]) : red[2 * t];
    bound[t] = m * sqrtf((float)D) * 1.01f;
  }
}

// Entry e of the rotary table: (cos, sin)(pos * omega_i) for i < half = D/2,
// in double, stored as float; omega_i = theta^(-2i/D), or the caller's
// inv_freq[i].
__device__ inline void rope_entry(float2 *tab, int32_t n_pos, int32_t half,
                                  double log_theta, const float *inv_freq,
                                  int64_t e) {
  if (e >= (int64_t)n_pos * half) return;
  const int32_t pos = (int32_t)(e / half), i = (int32_t)(e % half);
  const double freq =
      inv_freq ? (double)inv_freq[i]
               : exp(-(double)i / (double)half * log_theta);
  double sn, cs;
  sincos((double)pos * freq, &sn, &cs);
  tab[e] = make_float2((float)cs, (float)sn);
}

// First row of item `it` of a group of R rows from `base` cut into n_it items
// (its end: the first row of item it + 1).  Boundaries lie on multiples of
// 32 rows: near-equal items (the block kernels, which walk an item in
// passes), or, with exact_items, items of exactly rows_per_item rows and a
// shorter last one (the pass kernel serves an item in one pass, so no item
// may exceed it).
__device__ inline int64_t item_start(const PlanArgs &a, int64_t base, int64_t R,
                                     int64_t n_it, int64_t it) {
  if (it >= n_it) return base + R;
  return base + (a.exact_items ? it * a.rows_per_item
                               : (it * R / n_it) & ~(int64_t)31);
}

// What the work units' records need of the call.
struct UnitArgs {
  int32_t layer, n_rep;
  float c;  // softmax_scale * log2(e)
  int64_t ntok;
  const uint16_t *v;
};

// Work unit w of the pass kernel: item `it`, whose first pair's record is
// sp, for kv head g.  A unit whose logits the norm bounds cannot keep within
// the reference-free range (kNoRefBound) is marked by its pair's sign bit
// and left to the exact pass; its record holds one row and the first key of
// the pair, so that the pass kernel spends one batch of keys on it.  (Stored
// keys longer than the call's own gains allow: where the gains are over the
// bound themselves, all_over.)
__device__ inline void write_unit(const Plan &pl, const StoreView &sv,
                                  const UnitArgs &ua, int64_t w,
                                  const int4 &it, const int4 &sp, int32_t g) {
  const int D = sv.head_dim;
  const int32_t doc = pl.group_doc[it.x];
  const int32_t L = sv.doc_len[doc];
  const int64_t blk = sv.doc_off[doc];
  const float kb = fmaxf(
      pl.kown[0],
      sv.kmax[((int64_t)doc * sv.n_layers + ua.layer) * sv.n_kv_heads + g]);
  const bool over = ua.c * pl.kown[1] * kb * 1.001f > kNoRefBound;
  union {
    PassUnit u;
    int4 q[4];
  } r;
  auto put = [](int32_t *to, const uint16_t *p) {
    to[0] = (int32_t)(uint32_t)(uint64_t)p;
    to[1] = (int32_t)((uint64_t)p >> 32);
  };
  r.u.u0 = it.y / ua.n_rep;
  r.u.rows = (over ? 1 : it.z - it.y) | (it.y - r.u.u0 * ua.n_rep) << 8;
  r.u.s = over ? it.w | INT32_MIN : it.w;
  r.u.L = over ? 0 : L;
  put(r.u.k, sv.payload + k_offset(blk, L, sv.n_kv_heads, ua.layer, g, D));
  put(r.u.vt, sv.payload + vt_offset(blk, L, sv.n_kv_heads, ua.layer, g, D));
  put(r.u.own_k, pl.kh + (g * ua.ntok + sp.x) * D);
  put(r.u.own_v, ua.v + ((int64_t)sp.x * sv.n_kv_heads + g) * D);
  r.u.tok0 = sp.x;
  r.u.T = over ? 1 : sp.y;
  // (positions are stacked latest first: the item's latest position of its
  // first pair is at its first row)
  r.u.jmax = over ? 0 : sp.y - 1 - (it.y - sp.z) / ua.n_rep;
  r.u.g = g;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    reinterpret_cast<int4 *>(pl.units + w)[i] = r.q[i];
}

// Outputs of pair p, whose document is out of range or not resident: zeros
// and -inf LSE (the scheduler validated its token range), by one block.
// With no token ranges (score mode) pair p owns row p; out may then be NULL.
__device__ inline void zero_pair(int32_t p, const int32_t *cu, int32_t Hq,
                                 int32_t D, uint16_t *out, float *lse) {
  const int64_t t0 = cu ? cu[p] : p, t1 = cu ? cu[p + 1] : p + 1;
  const int64_t n16 = (t1 - t0) * Hq * D / 8;
  uint4 *o = reinterpret_cast<uint4 *>(out + t0 * Hq * D);
  if (out)
    for (int64_t e = threadIdx.x; e < n16; e += blockDim.x)
      o[e] = make_uint4(0, 0, 0, 0);
  if (lse)
    for (int64_t e = threadIdx.x; e < (t1 - t0) * Hq; e += blockDim.x)
      lse[t0 * Hq + e] = -INFINITY;
}

// score_only: one stacked token per pair (its score token, the last one)
// instead of all T_p.
struct PlanShape {
  int32_t n_pairs, n_rep, max_tokens, rows_per_item;
  int64_t n_docs, total_tokens;
  int32_t max_len, n_kv_heads;
  int32_t head_dim = kHeadDim;
  bool score_only = false;
  bool stream = false;  // the pass kernel runs: room for k^ of every token
                        // and the work-unit table
};

size_t plan_bytes(const PlanShape &s);
Plan plan_carve(void *ws, const PlanShape &s);
int64_t *plan_totals(const Plan &pl);
int32_t *plan_next(const Plan &pl);

// Batches of up to this many pairs are planned by plan.hip.
constexpr int kPlanPairs = 8192;
inline bool plan_is_small(const PlanShape &s) {
  return s.n_pairs <= kPlanPairs;
}

// Launchers (return hipError_t of the last launch).
hipError_t launch_store_put(const dopr_store &st, int32_t layer, int64_t n,
                            const int32_t *doc_ids, const int64_t *src_cu,
                            const uint16_t *k, const uint16_t *v,
                            hipStream_t s);
hipError_t launch_gather(const dopr_store &st, int32_t layer, int32_t n,
                         const int32_t *doc_ids, const int64_t *out_cu,
                         uint16_t *k, uint16_t *v, hipStream_t s);
hipError_t launch_store_copy(const dopr_store &dst, const dopr_store &src,
                             hipStream_t s);

struct AttnCall {
  const dopr_store *st;
  int32_t layer;
  const dopr_attn_args_t *a;
  int32_t n_rep;
  const dopr_score_head_t *head = nullptr;  // score mode (last layer)
};
// group.hip: the rotary table, a launch of its own.
hipError_t launch_rope_table(const AttnCall &c, const Plan &pl, hipStream_t s);
// plan.hip: the plan of a small batch, and (with k^ where the pass kernel
// runs, and the zero outputs of pairs without a document) its tables.
hipError_t launch_plan_one(const AttnCall &c, const Plan &plan,
                           const PlanShape &shape, const PlanArgs &pa,
                           int64_t lpt_units, hipStream_t s);
hipError_t launch_plan_fill(const AttnCall &c, const Plan &plan,
                            const PlanShape &shape, const PlanArgs &pa,
                            hipStream_t s);
inline UnitArgs unit_args(const AttnCall &c) {
  return {c.layer, c.n_rep, c.a->softmax_scale * 1.4426950408889634f,
          c.a->total_tokens, static_cast<const uint16_t *>(c.a->v)};
}
hipError_t launch_plan(const AttnCall &c, const Plan &plan,
                       const PlanShape &shape, hipStream_t s);
hipError_t launch_attention(const AttnCall &c, const Plan &plan,
                            const PlanShape &shape, hipStream_t s);
hipError_t launch_score(const dopr_score_args_t *a, hipStream_t s);
// width: the score head's input width, n_q_heads * head_dim.
hipError_t launch_score_reduce(const Plan &pl, int32_t n_pairs, int32_t n_q_heads,
                               int32_t width, const dopr_score_head_t *head,
                               hipStream_t s);

// ---------------------------------------------------------------------------
// Decoder layer around the attention (layer.hip).
constexpr int64_t kMlpChunk = 32768;               // MLP tokens per chunk
constexpr size_t kGemmWorkspace = size_t(64) << 20;  // hipBLASLt workspace

struct LayerShape {
  int64_t ntok;
  int32_t hidden, inter, hq, hkv;
};

struct LayerWs {
  uint16_t *h;    // [Ntok][W]   RMSNorm(x), later RMSNorm(x2)
  uint16_t *q;    // [Ntok][Hq][D]
  uint16_t *k;    // [Ntok][Hkv][D]
  uint16_t *v;    // [Ntok][Hkv][D]
  uint16_t *att;  // [Ntok][Hq][D] attention rows
  uint16_t *gu;   // [chunk][2I]  gate | up
  uint16_t *act;  // [chunk][I]   SiLU(gate) * up
  void *gemm_ws;
  size_t gemm_ws_bytes;
  int64_t chunk;
  void *plan;     // the attention plan follows the layer's buffers
  size_t bytes;   // layer buffers before the plan
};

LayerWs layer_carve(void *base, const LayerShape &s);
// Return 0, -1 for a HIP launch error, or a hipBLASLt status.
int launch_layer_pre(const LayerShape &s, const dopr_layer_args_t *l,
                     const LayerWs &w, float eps, hipStream_t st);
int launch_layer_post(const LayerShape &s, const dopr_layer_args_t *l,
                      const LayerWs &w, float eps, hipStream_t st);
const char *gemm_status_str(int s);

// Offline salience selection (salience.hip).
constexpr int kSalienceMaxLen = 4096;   // longest document (keys in LDS)
constexpr int kSalienceMaxP = 64;       // largest top-p (register list bound)
constexpr size_t kSalienceAbarBudget = size_t(1) << 30;  // scratch bytes

struct SalienceParams {
  const uint16_t *q, *k;     // [Ntok, Hq, D], [Ntok, Hkv, D]
  const int32_t *cu;         // [n_docs + 1]
  int32_t n_docs, d0;        // all docs; first doc of this launch
  int32_t hq, hkv, n_rep, max_len, top_p;
  int64_t total_tokens;
  float c;                   // softmax_scale * log2(e)
  float inv_hq;
  float *lse2;               // [Hq][Ntok] log2-domain row log-sum-exp
  float *kmax;               // [n_docs][Hkv][kKeyNormParts] partial maxima
                             // of the key norms per document
  float *abar;               // doc d - d0 at (d - d0) * abar_stride
  int64_t abar_stride;       // max_len * max_len
  float *u;                  // [Ntok]
  int32_t *status;           // deferred error word, or NULL
};

struct TopkParams {
  const int32_t *cu, *cs;    // [n_docs + 1] token and selection offsets
  const float *u;
  int32_t *selected;
  int32_t max_len;
  int64_t total_tokens, total_select;
  int32_t *status;
};

hipError_t launch_salience_check(const SalienceParams &p, hipStream_t s);
hipError_t launch_key_norms(const SalienceParams &p, hipStream_t s);
constexpr int kKeyNormParts = 8;  // partial maxima per (document, kv head)
hipError_t launch_salience_chunk(const SalienceParams &p, int32_t n_docs,
                                 int hr, int pm, hipStream_t s);
hipError_t launch_topk(const TopkParams &p, int32_t n_docs, hipStream_t s);

// Record a deferred error code in a status word (first error wins).
__device__ inline void raise_status(int32_t *status, int32_t code) {
  atomicCAS(status, 0, code);
}

}  // namespace dopr
