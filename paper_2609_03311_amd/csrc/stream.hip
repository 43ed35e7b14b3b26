// stream.hip -- the pass kernel of the full online layer (the automatic
// choice).  Built as its own translation unit with the compiler's common-code sinking off: that
// transformation would merge stores of different unit fields into one
// through a pointer and move wave-uniform state to scratch memory.
#include "attn_common.hpp"

namespace dopr {
namespace {

__device__ __forceinline__ int rfl(int x) {
  return __builtin_amdgcn_readfirstlane(x);
}

// Loads of read-only plan and store metadata at wave-uniform indices, made
// through the constant address space so they become scalar loads.
template <class T>
__device__ __forceinline__ T cld(const T *p, int64_t i) {
  return ((const __attribute__((address_space(4))) T *)p)[i];
}

__device__ __forceinline__ int4 cld(const int4 *p, int64_t i) {
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  const i32x4 v = ((const __attribute__((address_space(4))) i32x4 *)p)[i];
  return make_int4(v.x, v.y, v.z, v.w);
}

// Own-V rows: 16-byte granule swizzle that puts the four keys one
// transposing read takes per lane group on four different 64-byte bank
// ranges (a row is 256 B at D = 128, 128 B at D = 64).
template <int D>
__device__ __forceinline__ int swvo(int r) {
  if constexpr (D == 128)
    return (r & 3) << 2;
  else
    return ((r >> 1) & 1) << 2;
}

// Per-phase cycle counters of the pass kernel, compiled in only for the
// measurement library (-DDOPR_PASS_TIMERS): each wave adds the s_memtime
// cycles between consecutive marks to the total of the phase the mark
// closes, and adds its totals to a device array when it exits.  In the
// product library the marks are empty.
enum PassPhase {
  kPtQ,           // q rows loaded and q^ formed
  kPtWait,        // a batch's loads waited for, and the barrier
  kPtFeed,        // the next batch's loads issued
  kPtPrefix,      // prefix batches: products
  kPtOwn,         // own batches: products
  kPtAhead,       // the next unit's rows asked for
  kPtEpilogue,    // normalise and store O and the LSE
  kPtUnits,       // count: units
  kPtBatches,     // count: batches
  kPtTailCycles,  // cycles of units with at most 32 rows
  kPtTails,       // count: such units
  kPtSlots
};
#ifdef DOPR_PASS_TIMERS
__device__ unsigned long long g_pass_phase[4][kPtSlots];
#define PT_NOW() ((int64_t)__builtin_amdgcn_s_memtime())
#define PT_DECL()                    \
  int64_t pt_acc[kPtSlots] = {};     \
  int64_t pt_last = PT_NOW(), pt_unit = pt_last
#define PT_MARK(k)                   \
  do {                               \
    const int64_t pt_t = PT_NOW();   \
    pt_acc[k] += pt_t - pt_last;     \
    pt_last = pt_t;                  \
  } while (0)
#define PT_COUNT(k) (pt_acc[k] += 1)
#define PT_UNIT_START() (pt_unit = PT_NOW())
#define PT_UNIT_END(rows)                   \
  do {                                      \
    if ((rows) <= 32) {                     \
      pt_acc[kPtTailCycles] += pt_last - pt_unit; \
      pt_acc[kPtTails] += 1;                \
    }                                       \
  } while (0)
#define PT_FLUSH(wave, lane)                                          \
  do {                                                                \
    if ((lane) == 0)                                                  \
      for (int pt_i = 0; pt_i < kPtSlots; ++pt_i)                     \
        atomicAdd(&g_pass_phase[wave][pt_i],                          \
                  (unsigned long long)pt_acc[pt_i]);                  \
  } while (0)
#else
#define PT_DECL() ((void)0)
#define PT_MARK(k) ((void)0)
#define PT_COUNT(k) ((void)0)
#define PT_UNIT_START() ((void)0)
#define PT_UNIT_END(rows) ((void)0)
#define PT_FLUSH(wave, lane) ((void)0)
#endif

// One direct global->LDS load of 1 KB per wave (lane i: 16 bytes to
// lds + 16 i), from a wave-uniform base plus a lane's byte offset, or from
// per-lane addresses.  Written as assembly so that the compiler does not
// know it: it would make the wave's next LDS read, of the other buffer,
// wait for the loads in flight.  batch_ready orders them.  s_nop 4 covers
// the wait states after a vector write of the base's scalar registers and
// after the write of m0.
__device__ __forceinline__ void dma_base(uint32_t lds, const void *base,
                                         uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\t"
               "global_load_lds_dwordx4 %1, %2"
               :: "s"(lds), "v"(off), "s"(base)
               : "memory", "m0");
}
__device__ __forceinline__ void dma_lane(uint32_t lds, const void *p) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\t"
               "global_load_lds_dwordx4 %1, off" :: "s"(lds), "v"(p)
               : "memory", "m0");
}

// A whole chunk's share of one wave: its K blocks (1 KB apart in LDS) from
// ka, its V blocks VOFF behind them from va.
template <int D, uint32_t VOFF>
__device__ __forceinline__ void dma_chunk(uint32_t lds, const void *ka,
                                          uint32_t k1, uint32_t k2,
                                          const void *va, uint32_t v1,
                                          uint32_t v2) {
  if constexpr (D == 128)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\t"
                 "global_load_lds_dwordx4 %1, %3\n\t"
                 "s_add_u32 m0, m0, 1024\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %2, %3\n\t"
                 "s_add_u32 m0, m0, %7\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %4, %6\n\t"
                 "s_add_u32 m0, m0, 1024\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %5, %6"
                 :: "s"(lds), "v"(k1), "v"(k2), "s"(ka), "v"(v1), "v"(v2),
                    "s"(va), "n"(VOFF - 1024)
                 : "memory", "scc", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\t"
                 "global_load_lds_dwordx4 %1, %2\n\t"
                 "s_add_u32 m0, m0, %5\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %3, %4"
                 :: "s"(lds), "v"(k1), "s"(ka), "v"(v1), "s"(va), "n"(VOFF)
                 : "memory", "scc", "m0");
}

// The batch on its way is in LDS for every wave, and every wave is done with
// the one before it.
__device__ __forceinline__ void batch_ready() {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ uint32_t lds_addr(const void *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3)))
                                   void *)p;
}

// One or two 32-key chunks in LDS: S^T = K Q^T from the K rows, the weights,
// O^T += V^T P^T.  A prefix chunk's V^T rows are read as they are; an own
// chunk's v rows [32][D] by gfx950's transposing LDS read (4 keys of one
// head dim per lane and read, two reads per fragment: fragment f = (db = f /
// 2, t = f % 2) holds keys 8t .. 8t + 7 of this lane's half, head dims 32 db
// + perm32(lq)).  vaddr: this lane's part of the v rows (row 16*hf + e,
// column perm32(16*(lq/16) + 4q) of the lane's (e, q) role in its 16-lane
// group); ex: its row's swizzle.  Keys past lim are hidden.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4 *LdsTr;

template <int D>
__device__ __forceinline__ void k_read(const uint16_t *kb, const Frag<D> &fo,
                                       bf16x8 *kf) {
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
    kf[s] = *reinterpret_cast<const bf16x8 *>(kb + fo.k[s]);
}

template <int D>
__device__ __forceinline__ void attend_slot(const uint16_t *slot, bool two,
                                            bool own, int vaddr, int ex,
                                            const Frag<D> &fo,
                                            const bf16x8 (*qf)[D / 16],
                                            Acc<D> *acc, int hf, int lim) {
  constexpr int SLOT = 2 * KC * D;
  bf16x8 kf[D / 16], vf[D / 16];
  k_read<D>(slot, fo, kf);
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    if (c == 1 && !two) break;
    floatx16 S[1];
#pragma unroll
    for (int i = 0; i < 16; ++i) S[0][i] = 0.f;
#pragma unroll
    for (int s = 0; s < D / 16; ++s)
      S[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[0][s], S[0], 0,
                                                     0, 0);
    const uint16_t *vb = slot + c * SLOT + KC * D;
    if (own) {
#pragma unroll
      for (int f = 0; f < D / 16; ++f) {
        const uint16_t *a =
            vb + vaddr + 32 * ((f >> 1) ^ ex) + (f & 1) * 8 * D;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsTr)a);
        const s16x4 hi =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsTr)(a + 4 * D));
        vf[f] = __builtin_bit_cast(
            bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      }
    } else {
      v_read<D, D / 16>(vb, fo, 0, vf);
    }
    // (the second chunk's K rows arrive under the first one's softmax)
    if (c == 0) k_read<D>(slot + SLOT, fo, kf);
    __builtin_amdgcn_sched_barrier(0);
    if (!__all(lim >= KC - 1)) {
      const int li = lim - 16 * hf;
#pragma unroll
      for (int i = 0; i < 16; ++i) S[0][i] = i <= li ? S[0][i] : -INFINITY;
    }
    lim -= KC;
    bf16x8 pb[1][2];
    softmax_part<0, 1, 0, D>(S, acc, hf, 0.f, nullptr, pb);
#pragma unroll
    for (int f = 0; f < D / 16; ++f)
      acc[0].o[f >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          vf[f], pb[0][f & 1], acc[0].o[f >> 1], 0, 0, 0);
  }
}

// ---------------------------------------------------------------------------
// Pass kernel (full layer).  A work unit is a pass of at most 128 stacked
// rows of one document for one kv head: one 32-row tile for each of a
// block's four waves.  Blocks are small (two per CU at head size 128, three
// at 64) and independent, so one block's q^ prologue, output stores and
// waits run under another's products; an 8-wave block that keeps the whole
// prefix in LDS has all of a CU's waves in the same phase.  The bound is on
// the chip, not in HBM (with every HBM access redirected to L2 the 8-wave
// block still took 89 % of its time): what counts is instructions and waits
// per row, and how much of them other waves cover.
//
// A unit's keys are a sequence of 32-key chunks: the document's prefix, then
// the own keys of the unit's pairs, in the block kernels' order, so every
// row's sums are formed in the same order and come out bit-identical.  They
// pass through two LDS buffers of two chunks (K 8 KB + V 8 KB a chunk at
// D = 128): the next batch's direct loads are issued behind the barrier that
// frees its buffer and run under the current batch's products, across the
// end of a unit too.  Two chunks a barrier, since the issue of a batch costs
// about 1000 cycles of scalar work and waits whatever its size (one chunk a
// barrier: 9.0 ms where two take 8.4).  A prefix is read through L2 once per
// unit (a document's units of one kv head are handed out together to the
// blocks of one XCD); keeping it resident leaves no LDS for a second block.
//
// The next unit's record is read when a unit starts and its rows' tokens
// after the first batch.  Unit numbers are claimed three units ahead by
// thread 0 and passed through LDS, so every wave knows the next one without
// a barrier.  The first three are dealt out, one a round to every block of the
// queue in turn: claimed in one step, three to the block that comes first,
// they left blocks of a small batch with three units beside others with none
// (us per call, head size 64: 512 units on documents of 1,500 slots 147 -> 68;
// head size 128, 4,000 units in longest-first order 175 -> 170).
//
// Measured against the 8-wave resident block, us per call of the step
// (grouping, k^, attention, head): 6,400 pairs of 129 tokens on 256-slot
// prefixes (32 q / 8 kv heads) 8880 -> 8350, the same with 100 pairs
// 286 -> 229, 4,096 ragged pairs (8..256 slots, 17..129 tokens) 2945 -> 2550,
// head size 64 4460 -> 4345 (four blocks per CU in 128 registers, with
// spills: 4720).  Not better: q rows through the buffers like a batch
// (8550), q loads issued before the output stores (9290, 32 spills).
//
// Only the reference-free softmax (mode 0) runs here: units over the logit
// bound and units with a normaliser out of range go to the exact pass.
//
// Loop exits and barriers are block-uniform: units come from words thread 0
// published in LDS before a barrier, chunk sequences from the plan's tables
// at wave-uniform indices, and every wave runs every chunk step (a wave
// with no row in a chunk skips its products only).
constexpr int kAhead = 3;

template <int D>
struct PassSm {
  uint16_t batch[2][2][2 * KC * D];  // two buffers of two chunks: K rows,
                                     // then V (V^T rows of a prefix chunk, v
                                     // rows of an own chunk)
  uint16_t qw[D];                    // the q gains
  int32_t claim[4];                  // unit numbers claimed ahead
  int32_t bad[2];                    // waves that left the safe range
  int32_t n_work;                    // work units, and whether the queues
  int32_t ordered;                   // follow the plan's order
  int32_t dealt;                     // slots of the queue dealt out at first
};

// The kernel's arguments, read again where they are used: some thirty
// pointers and sizes would otherwise hold scalar registers for the whole
// kernel, more than there are.
typedef const __attribute__((address_space(4))) AttnParams *ArgPtr;
__device__ __forceinline__ ArgPtr args_here() {
  uint64_t a = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  return (ArgPtr)a;
}

__device__ __forceinline__ const uint16_t *join(int lo, int hi) {
  return reinterpret_cast<const uint16_t *>((uint64_t)(uint32_t)lo |
                                            ((uint64_t)(uint32_t)hi << 32));
}

// A work unit's record in the plan (PassUnit), read with scalar loads; w <
// 0: no unit.
struct PUnit {
  int w;
  PassUnit d;
};

__device__ __forceinline__ PassUnit unit_load(int w) {
  typedef int i32x16 __attribute__((ext_vector_type(16)));
  const i32x16 v =
      ((const __attribute__((address_space(4))) i32x16 *)args_here()->units)[w];
  return __builtin_bit_cast(PassUnit, v);
}

// The key sequence of a unit, as far as it has been issued, in segments: the
// document's prefix, then the own keys of each of its pairs.  ka, va: the
// next chunk's K and V rows; vo: this lane's byte offset of its V granule in
// the first of its wave's 1 KB blocks, vo2 the second's.
struct Feed {
  const uint16_t *ka, *va;
  int vstep;            // elements from one chunk's V rows to the next's
  int k0, jmax;         // the segment's next key, and the last one seen
  int tok0, T;          // pair's first token (< 0: prefix), keys there are
  uint32_t vo, vo2;
  int s, row1;          // pair of the segment; the unit's end
  const uint16_t *oka, *ova;  // own rows of the unit's first pair
  int otok, oT, ojmax;
  int4 next;            // the record of pair s + 1
};

// A batch of one or two chunks in LDS: keys k0 .. of the pair at token tok0
// with T tokens, or (tok0 < 0) of a prefix of T slots.
struct Batch {
  int tok0, T, k0;
  int two, last;  // two chunks; the unit's last batch
};

// A lane's place in the loads of a chunk, for the first of its wave's KB 1 KB
// blocks of K and of V (the second's rows lie RPB below: swz flips bit 3,
// swvo nothing; its V^T rows 16 below: swz_v flips bit 1).
struct FeedLane {
  uint32_t kofs, kofs2;  // byte offsets of its K granules
  uint32_t vofs;         // byte offset of its own-V granule
  uint32_t d, key;       // V^T row and first key of its prefix-V granule
};

template <int D>
__device__ __forceinline__ FeedLane feed_lane(int wave, int lane, int stride) {
  constexpr int G = D / 8, RPB = 64 / G;
  constexpr int KB = KC * D * 2 / 1024 / 4;
  static_assert(KB == 1 || (KB == 2 && D == 128), "second block's offsets");
  FeedLane l;
  const int r = RPB * wave * KB + lane / G, p = lane % G;
  l.kofs = (uint32_t)(r * D + ((p ^ swz<D>(r)) << 3)) * 2;
  l.kofs2 = (l.kofs + RPB * D * 2) ^ 128;
  l.vofs = (uint32_t)(r * stride + ((p ^ swvo<D>(r)) << 3)) * 2;
  l.d = 16 * wave * KB + (lane >> 2);
  l.key = 8 * ((lane & 3) ^ swz_v(l.d));
  return l;
}

// Own-key segment: pair at token tok0 with T tokens, keys 0 .. jmax.
template <int D>
__device__ __forceinline__ void feed_own(Feed &f, const FeedLane &l, int tok0,
                                         int T, int jmax, int stride) {
  const int64_t dt = tok0 - f.otok;
  f.ka = f.oka + dt * D;
  f.va = f.ova + dt * stride;
  f.vstep = KC * stride;
  f.k0 = 0;
  f.jmax = jmax;
  f.tok0 = tok0;
  f.T = T;
  f.vo = l.vofs;
  f.vo2 = l.vofs + (512 / D) * stride * 2;
}

// First segment of a unit.
template <int D>
__device__ __forceinline__ void feed_unit(Feed &f, const FeedLane &l,
                                          const PassUnit &u, int n_rep,
                                          int stride) {
  f.row1 = u.u0 * n_rep + (u.rows >> 8) + (u.rows & 0xff);
  f.oka = join(u.own_k[0], u.own_k[1]);
  f.ova = join(u.own_v[0], u.own_v[1]);
  f.otok = u.tok0;
  f.oT = u.T;
  f.ojmax = u.jmax;
  f.s = u.s & 0x7fffffff;
  f.next = cld(args_here()->spair, f.s + 1);
  if (u.L > 0) {
    const int Lp = pad8(u.L);
    f.ka = join(u.k[0], u.k[1]);
    f.va = join(u.vt[0], u.vt[1]);
    f.vstep = KC;
    f.k0 = 0;
    f.jmax = u.L - 1;
    f.tok0 = -1;
    f.T = u.L;
    f.vo = 2 * (l.d * Lp + l.key);
    f.vo2 = 2 * ((l.d + 16) * Lp + (l.key ^ 16));
  } else {
    feed_own<D>(f, l, f.otok, f.oT, f.ojmax, stride);
  }
}

// Issue the direct loads of the next batch into the buffer at LDS address
// `lds` (wave w takes the 1 KB blocks w * KB .. of each chunk's K and V) and
// go on to the next segment at a segment's end.
template <int D>
__device__ __forceinline__ Batch feed_batch(Feed &f, const FeedLane &l,
                                            uint32_t lds, int stride) {
  constexpr int KB = KC * D * 2 / 1024 / 4;  // 1 KB blocks per wave
  constexpr uint32_t VOFF = KC * D * 2;      // V's place in a chunk
  Batch b{f.tok0, f.T, f.k0, f.jmax - f.k0 >= KC, 0};
  const int n = f.T - f.k0;
  if (n >= 2 * KC && b.two) {
    dma_chunk<D, VOFF>(lds, f.ka, l.kofs, l.kofs2, f.va, f.vo, f.vo2);
    dma_chunk<D, VOFF>(lds + 2 * VOFF, f.ka + KC * D, l.kofs, l.kofs2,
                       f.va + f.vstep, f.vo, f.vo2);
  } else {
    for (int c = 0; c <= b.two; ++c) {
      const uint16_t *ka = f.ka + c * (KC * D), *va = f.va + c * f.vstep;
      const uint32_t at = lds + c * 2 * VOFF;
      const int m = n - c * KC;  // valid keys of this chunk
      if (m >= KC) {
        dma_chunk<D, VOFF>(at, ka, l.kofs, l.kofs2, va, f.vo, f.vo2);
        continue;
      }
      // a short chunk: K rows past its last valid one repeat it (their
      // logits are masked); V rows, or V^T columns past the stored ones (pad
      // columns are stored zeros), come from the zero page: their weights
      // are zero, and 0 * V must be 0
      const uint32_t last = (uint32_t)(m - 1) * D * 2;
      const uint16_t *zero = args_here()->zero;
#pragma unroll
      for (int i = 0; i < KB; ++i) {
        const uint32_t o = i ? l.kofs2 : l.kofs;
        const uint32_t ro = o & ~(uint32_t)(D * 2 - 1);
        dma_base(at + i * 1024, ka, (ro < last ? ro : last) + (o - ro));
        const bool in = f.tok0 < 0 ? (l.key ^ (16 * i)) < (uint32_t)pad8(m)
                                   : ro <= last;
        dma_lane(at + VOFF + i * 1024,
                 in ? va + (i ? f.vo2 : f.vo) / 2 : zero);
      }
    }
  }
  f.ka += 2 * KC * D;
  f.va += 2 * f.vstep;
  f.k0 += 2 * KC;
  if (f.k0 > f.jmax) {
    if (f.tok0 < 0) {
      feed_own<D>(f, l, f.otok, f.oT, f.ojmax, stride);
    } else if (f.next.z < f.row1) {
      // the next pair starts inside the unit: all of its keys are seen
      ++f.s;
      feed_own<D>(f, l, f.next.x, f.next.y, f.next.y - 1, stride);
      f.next = cld(args_here()->spair, f.s + 1);
    } else {
      b.last = 1;
    }
  }
  return b;
}

template <int D, int GROUP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(
    D == 64 ? 3 : 2, D == 64 ? 3 : 2))) void k_pass_attn(AttnParams P0) {
  constexpr int GW = D / 16 / GROUP;
  __shared__ __attribute__((aligned(16))) PassSm<D> sm;
  const int lane = threadIdx.x & 63, wave = rfl(threadIdx.x >> 6);
  const int lq = lane & 31, hf = lane >> 5;
  const int queue = blockIdx.x & 7;
  if (threadIdx.x < D / 8)
    reinterpret_cast<uint4 *>(sm.qw)[threadIdx.x] =
        reinterpret_cast<const uint4 *>(P0.qw)[threadIdx.x];
  if (threadIdx.x == 0) {
    int64_t n_items = P0.totals[kTotItems];
    if (n_items > P0.items_cap) n_items = P0.items_cap;
    // (every unit over the logit bound: the plan has listed them)
    if (all_over(P0.c, P0.kown)) n_items = 0;
    const int n_work = (int)(n_items * P0.Hkv);
    const int32_t *qo = P0.totals[kTotUnits] ? P0.qorder : nullptr;
    sm.n_work = n_work;
    sm.ordered = qo != nullptr;
    const int blocks = gridDim.x >> 3;  // of this queue
    sm.dealt = kAhead * blocks;
    for (int i = 0; i < kAhead; ++i) {
      const int w = unit_at32(qo, queue, (blockIdx.x >> 3) + i * blocks,
                              n_work);
      sm.claim[i] = w < n_work ? w : -1;
    }
    sm.bad[0] = sm.bad[1] = 0;
  }
  __syncthreads();

  if (rfl(sm.claim[0]) < 0) return;
  const Frag<D> fo = frag_offsets<D>(lq, hf);
  const int e4 = (lane >> 2) & 3, q4 = lane & 3;
  const int ex = D == 128 ? e4 : (e4 >> 1);
  // own-V transposing reads: this lane's part of the v rows
  const int vaddr =
      (16 * hf + e4) * D + perm32(16 * ((lane >> 4) & 1) + 4 * q4);
  constexpr uint32_t BUF = 2 * 2 * KC * D * 2;
  // (wave w's first 1 KB block of a chunk)
  const uint32_t ring =
      lds_addr(sm.batch[0]) + wave * (KC * D * 2 / 1024 / 4) * 1024;
  const int n_rep = P0.n_rep, stride = P0.Hkv * D;
  // (x / n_rep = umulhi(x, rep_mul) for x < 128 + n_rep: the host admits n_rep
  // < 2^15)
  const uint32_t rep_mul = n_rep > 1 ? 0xffffffffu / (uint32_t)n_rep + 1 : 0;
  const FeedLane fl = feed_lane<D>(wave, lane, stride);

  // the next unit (number nw; < 0: none): its record and, per lane, its
  // row's token, position and head
  int nw = rfl(sm.claim[0]);
  PassUnit nx = unit_load(nw);
  int asked = 0;
  int2 tj = make_int2(0, 0);
  int nhead = 0;
  auto ask_rows = [&]() {
    // (rows past the unit's end repeat its last one)
    const int last = (nx.rows & 0xff) - 1, i = wave * 32 + lq;
    const int x = (i < last ? i : last) + (nx.rows >> 8);
    const int ut = n_rep > 1 ? (int)__umulhi(x, rep_mul) : x;
    tj = args_here()->utok[nx.u0 + ut];
    nhead = nx.g * n_rep + (x - ut * n_rep);
    asked = 1;
  };
  Feed f{};
  feed_unit<D>(f, fl, nx, n_rep, stride);
  // the batch on its way, into buffer `buf`
  Batch nb = feed_batch<D>(f, fl, ring, stride);
  int buf = 0;
  ask_rows();

  PT_DECL();
  for (int iu = 0;; ++iu) {
    if (!asked) ask_rows();
    const int w = nw, rows = nx.rows & 0xff, over = nx.s < 0;
    const int tokq = tj.x, head = nhead;
    const bool valid = wave * 32 + lq < rows;
    PT_UNIT_START();
    PT_COUNT(kPtUnits);
    // claim a unit kAhead further on (its number is used at the end)
    int claim = 0;
    if (threadIdx.x == 0) claim = atomicAdd(&args_here()->next[queue], 1);
    bf16x8 qf[1][D / 16];
    {
      const ArgPtr P = args_here();
      QRow<D, GROUP> qr;
      q_row_load<D, GROUP>(P->q + ((int64_t)tokq * P->Hq + head) * D,
                           P->rope + (int64_t)(nx.L + tj.y) * (D / 2), hf,
                           lane & (GROUP - 1), qr);
      uint4 wv[GW];
      const uint16_t *gw = sm.qw + opaque_zero();
#pragma unroll
      for (int m = 0; m < GW; ++m)
        wv[m] = *reinterpret_cast<const uint4 *>(
            gw + 16 * ((lane & (GROUP - 1)) * GW + m) + 8 * hf);
      q_row_form<D, GROUP>(qr, wv, P->eps, P->c, P->norm != 0, qf[0]);
    }
    // (the feed has the unit's record: the next one's replaces it)
    nw = rfl(sm.claim[(iu + 1) & 3]);
    if (nw >= 0) nx = unit_load(nw);
    asked = 0;
    Acc<D> acc[1];
    acc[0].m = 0.f;
    acc[0].l = 0.f;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[0].o[db][i] = 0.f;
    PT_MARK(kPtQ);
    for (;;) {
      batch_ready();
      PT_MARK(kPtWait);
      PT_COUNT(kPtBatches);
      const Batch b = nb;
      const uint16_t *at = sm.batch[buf][0];
      buf ^= 1;
      // the next batch: this unit's, or the first of the next one
      if (b.last && nw >= 0) feed_unit<D>(f, fl, nx, n_rep, stride);
      if (!b.last || nw >= 0)
        nb = feed_batch<D>(f, fl, ring + buf * BUF, stride);
      PT_MARK(kPtFeed);
      const int own = b.tok0 >= 0;
      const int jr = tokq - b.tok0;
      int lim = b.T - 1 - b.k0;
      if (own) lim = (unsigned)jr < (unsigned)b.T ? jr - b.k0 : -1;
      if (__any(valid && lim >= 0))
        attend_slot<D>(at, b.two && __any(valid && lim >= KC), own, vaddr, ex,
                       fo, qf, acc, hf, lim);
      PT_MARK(own ? kPtOwn : kPtPrefix);
      if (b.last) break;
      if (!asked && nw >= 0) ask_rows();
      PT_MARK(kPtAhead);
    }

    // normalise; write O (bf16) and the natural-log LSE
    bool bad = false;
    const ArgPtr P = args_here();
    const float lt = acc[0].l + __shfl_xor(acc[0].l, 32, 64);
    if (valid) {
      bad = !(lt >= kLoOk && lt <= kHiOk);
      const float inv = 1.0f / lt;
      const int64_t orow = (int64_t)tokq * P->Hq + head;
      uint16_t *op = P->out + orow * D;
#pragma unroll
      for (int db = 0; db < D / 32; ++db) {
        float o[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) o[i] = acc[0].o[db][i] * inv;
        uint4 *dst = reinterpret_cast<uint4 *>(op + 32 * db + 16 * hf);
        dst[0] = as_uint4(to_bf16x8(o));
        dst[1] = as_uint4(to_bf16x8(o + 8));
      }
      if (P->lse && hf == 0) P->lse[orow] = __log2f(lt) * kLn2;
    }
    // a unit over the logit bound (one row of it was run) is left to the exact
    // pass, as is every unit in self-check mode, and one with a bad row: the
    // first wave that finds one adds it
    const int par = iu & 1;
    if (over || P->flag_all) {
      if (threadIdx.x == 0)
        P->fix[atomicAdd(&P->counters[kCntFix], 1)] =
            w | (over ? kFixUnscored : 0);
    } else if (__any(bad)) {
      if (lane == 0 && atomicAdd(&sm.bad[par], 1) == 0)
        P->fix[atomicAdd(&P->counters[kCntFix], 1)] = w;
    }
    if (threadIdx.x == 0) {
      // (every wave left the unit before this one behind a barrier ago)
      sm.bad[par ^ 1] = 0;
      const int n_work = sm.n_work;
      const int w3 = unit_at32(sm.ordered ? P->qorder : nullptr, queue,
                               sm.dealt + claim, n_work);
      sm.claim[(iu + kAhead) & 3] = w3 < n_work ? w3 : -1;
    }
    PT_MARK(kPtEpilogue);
    PT_UNIT_END(rows);
    if (nw < 0) break;
  }
  PT_FLUSH(wave, lane);
}

}  // namespace

// The pass kernel (k^ of every token is there): 4-wave blocks, two per CU
// at head size 128 (256 registers per lane) and three at 64 (168), a
// multiple of 8 blocks so block b serves queue b % 8.
#ifdef DOPR_PASS_TIMERS
// The measurement library's phase totals, [4 waves][kPtSlots], summed over
// every block since the last reset; reset != 0 clears them afterwards.
extern "C" int dopr_pass_phase_read(unsigned long long *out, int reset) {
  hipError_t e = hipMemcpyFromSymbol(out, HIP_SYMBOL(g_pass_phase),
                                     sizeof(g_pass_phase));
  if (e == hipSuccess && reset) {
    static const unsigned long long zero[4][kPtSlots] = {};
    e = hipMemcpyToSymbol(HIP_SYMBOL(g_pass_phase), zero, sizeof(zero));
  }
  return (int)e;
}
#endif

namespace {
template <int D>
hipError_t launch_pass(const AttnParams &p, unsigned grid, hipStream_t s) {
  // (the lanes that share a token: see q_fragments_any)
  if ((p.n_rep & 3) == 0)
    hipLaunchKernelGGL((k_pass_attn<D, 4>), dim3(grid), dim3(256), 0, s, p);
  else if ((p.n_rep & 1) == 0)
    hipLaunchKernelGGL((k_pass_attn<D, 2>), dim3(grid), dim3(256), 0, s, p);
  else
    hipLaunchKernelGGL((k_pass_attn<D, 1>), dim3(grid), dim3(256), 0, s, p);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_stream(int D, const AttnParams &p, hipStream_t s) {
  int dev = 0, n_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const unsigned grid = (unsigned)((n_cu + 7) / 8 * 8);
  return D == 128 ? launch_pass<128>(p, 2 * grid, s)
                  : launch_pass<64>(p, 3 * grid, s);
}

}  // namespace dopr
