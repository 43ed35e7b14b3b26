// salience.hip -- offline salience selection (Sec. 3.2.1, used by the
// offline compression of Sec. 3.3).
//
// For one document of n tokens with final-layer queries q^ [n, Hq, D] and
// keys k^ [n, Hkv, D] (as they enter the attention product):
//   A_h[j, i] = softmax_i(scale * q^_h[j] . k^_g[i]),  i <= j,  g = h / n_rep
//   Abar      = (1/Hq) sum_h A_h                     (rows attend, columns
//                                                      are attended)
//   u_i       = mean of the m = min(p, n - i) largest Abar[j, i], j >= i
//   selected  = the K positions with the largest u (ties: lower position),
//               written in ascending position order.
//
// Four kernels, each a plain pass over its data:
//   k_row_lse     per (row block of 128, kv head): the log2-domain
//                 log-sum-exp of every row of every q head of the group
//                 (scaled logits; one flash-style sweep over the visible
//                 keys with a running maximum).
//   k_mean_attn   per (row block, key block) of 128 x 128 on or below the
//                 diagonal: every head's probabilities exp2(S - lse2),
//                 summed over heads in head order, times 1/Hq, stored as
//                 fp32 row-major [n, n] (only i <= j is written).
// In both attention kernels the key blocks strictly below the diagonal,
// which every row of the block sees whole, take a path without masks or
// branches inside the head or sub-tile loops, in which one tile's products
// alternate with the exponentials of the tile before.  What bounds both is
// the issue of a 32 x 32 tile's 8 matrix and some 60 vector instructions
// (256 + 300 cycles, of which the chip overlaps a part) at a clock that the
// matrix power holds near 1.8 GHz; each fragment read feeds two tiles.
//   k_col_topp    per strip of 64 columns: each lane keeps the PM largest
//                 values of its column in a sorted register list while four
//                 waves (sixteen where the launch has few, long columns)
//                 stream interleaved rows; the lists are merged and the top m
//                 averaged.
//   k_topk        per document: radix search of the K-th largest u, then an
//                 ordered compaction of the chosen positions.
//
// Both attention kernels form S = K Q^T with the 32x32x16 bf16 MFMA in the
// same operand layout and the same k order, so the logits they see are the
// same fp32 values.  A-operand (key) rows are read in the order perm(m) so
// that lane half hf's 16 accumulators hold 16 consecutive keys 16 hf + i
// for the lane's query column.
#include <cmath>
#include <type_traits>

#include "internal.hpp"

namespace dopr {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int D = kHeadDim;
constexpr int kRowBlock = 128;   // rows per unit (4 waves x 32)
constexpr int kKeyBlock = 128;   // keys per mean-attention unit
constexpr int kStrip = 64;       // columns per top-p strip
// A strip's columns are split over sixteen waves instead of four where the
// launch has few strips and long columns: then a column's chain of loads is
// what it waits for.  With more strips the CUs are full either way, and the
// longer merge of sixteen lists costs more than the shorter chains save; the
// lists of more than 16 values merge too slowly for any split.  Whole call of
// 4 q and 4 kv heads, us, four -> sixteen waves.  Lists of 8: 256 strips of 512
// tokens 63.9 -> 60.8, of 1,000 91.4 -> 84.7, of 4,096 246 -> 207, 512 strips of
// 2,048 200 -> 196; 1,024 strips of 512 139 -> 148, of 2,048 370 -> 385.  Lists
// of 16: 192 strips of 1,536 tokens 119.6 -> 116.6, 256 of 4,096 259 -> 244; 256
// of 1,000 100.2 -> 101.3, 512 of 2,048 227 -> 243.  Lists of 32 (eight waves):
// 256 strips of 1,000 tokens 127.7 -> 131.7, of 4,096 315 -> 315.
struct ToppWide {
  int min_len;         // tokens from which on
  int64_t max_strips;  // strips of the launch up to which
};
constexpr ToppWide kToppWide8 = {512, 512}, kToppWide16 = {1024, 256};

__device__ __forceinline__ int perm(int m) {
  return ((m >> 2) & 1) * 16 + (m >> 3) * 4 + (m & 3);
}
// XOR swizzle of the 16-byte granules of a K row staged in LDS, so the rows
// read together by a quarter wave fall on distinct bank groups.
__device__ __forceinline__ int swz(int row) {
  return (row & 3) | ((row >> 2) & 4) | ((row << 1) & 8);
}

struct Doc {
  int64_t t0;
  int32_t n;
  bool ok;
};

__device__ __forceinline__ Doc doc_at(const SalienceParams &P, int d) {
  Doc r;
  const int32_t a = P.cu[d], b = P.cu[d + 1];
  r.t0 = a;
  r.n = b - a;
  r.ok = a >= 0 && r.n >= 1 && r.n <= P.max_len && b <= P.total_tokens;
  return r;
}

__device__ __forceinline__ bf16x8 ld8(const uint16_t *p) {
  return *reinterpret_cast<const bf16x8 *>(p);
}

// ---------------------------------------------------------------------------
// Keys are staged in LDS in blocks of 128 rows (32 KB), double-buffered so a
// block's direct global->LDS loads overlap the products on the previous one.
constexpr int kLdsK = kKeyBlock * D;  // bf16 elements (swizzled rows)

// Rows r0 .. r0+ROWS-1 of head h of the document in x [tokens, heads, D] (keys or
// queries) into `dst`: each lane writes 16 bytes of a 1 KB block (4 rows),
// fetching the global granule that the swizzled layout puts in its slot, so
// slot p of row r holds granule p ^ swz(r).  Rows past the document's end
// repeat row n-1.  Wave w takes the blocks w, w + 4, ...; a row 16 further on
// flips bit 2 of swz.  r0 and h are wave-uniform.  The loads are written as
// assembly so that the compiler does not know them: it would make the next
// LDS read, of the other buffer, wait for the loads in flight.  wait_vmem and
// the barrier behind it order them.  s_nop 4 covers the wait states after the
// writes of the base's scalar registers and of m0.  A row's byte offset from
// the block's first is kept in 32 bits, which 127 rows of up to kOffsetHeads
// heads fit; rows of more heads (WIDE) are loaded through full addresses, in
// kernels of their own (a branch here cost the others 0.3 to 0.9 %).
constexpr int kOffsetHeads = 1 << 17;

template <bool WIDE, int ROWS = kKeyBlock>
__device__ __forceinline__ void stage_rows(const uint16_t *x, int heads,
                                           const Doc &doc, int r0, int h,
                                           uint16_t *dst) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lds = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)dst);
  const uint16_t *base = x + ((doc.t0 + r0) * heads + h) * D;
  const int last = doc.n - 1 - r0;
  int row = 4 * wave + (lane >> 4);
  // (computed here each time: kept, the eight offsets would take registers)
  asm volatile("" : "+v"(row));
  const uint32_t gran = ((lane & 15) ^ swz(row)) * 16;
  if (WIDE) {
#pragma unroll 1
    for (int i = 0; i < ROWS / 16; ++i) {
      const uint16_t *p =
          base + (int64_t)min(row + 16 * i, last) * heads * D +
          ((gran ^ (i & 1 ? 64u : 0u)) >> 1);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\t"
                   "global_load_lds_dwordx4 %1, off"
                   :: "s"(lds + (wave + 4 * i) * 1024), "v"(p)
                   : "memory", "m0");
    }
    return;
  }
  const uint32_t stride = (uint32_t)(heads * D * 2);
  if (last >= ROWS - 1) {
    const uint32_t even = (uint32_t)row * stride + gran;
    const uint32_t odd = even ^ 64u;
#pragma unroll
    for (int i = 0; i < ROWS / 16; ++i)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\t"
                   "global_load_lds_dwordx4 %1, %2"
                   :: "s"(lds + (wave + 4 * i) * 1024),
                      "v"(i & 1 ? odd : even),
                      "s"(base + (int64_t)i * 16 * heads * D)
                   : "memory", "m0");
    return;
  }
#pragma unroll
  for (int i = 0; i < ROWS / 16; ++i) {
    const uint32_t off = (uint32_t)min(row + 16 * i, last) * stride +
                         (gran ^ (i & 1 ? 64u : 0u));
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\t"
                 "global_load_lds_dwordx4 %1, %2"
                 :: "s"(lds + (wave + 4 * i) * 1024), "v"(off), "s"(base)
                 : "memory", "m0");
  }
}

__device__ __forceinline__ void wait_vmem() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// A lane's operand fragments of 32-row tile t of a staged block: row `r` of
// the tile (perm(lq) for a product's key operand, lq for its q operand), lane
// half hf.
__device__ __forceinline__ bf16x8 row_frag(const uint16_t *buf, int t, int r,
                                           int hf, int s) {
  const int row = 32 * t + r;
  return ld8(buf + row * D + (((2 * s + hf) ^ swz(row)) << 3));
}
__device__ __forceinline__ void row_frags(const uint16_t *buf, int t, int r,
                                          int hf, bf16x8 (&f)[8]) {
#pragma unroll
  for (int s = 0; s < 8; ++s) f[s] = row_frag(buf, t, r, hf, s);
}

// ---------------------------------------------------------------------------
// Largest key norm of each (document, kv head), as kKeyNormParts partial
// maxima over interleaved 64-row slices.  grid (docs, kv heads, parts);
// 16 lanes per key row (16 bytes each), four rows per wave and step, four
// steps in flight.
__global__ __launch_bounds__(256) void k_key_norm(SalienceParams P) {
  __shared__ float wmax[4];
  const int d = blockIdx.x, g = blockIdx.y, part = blockIdx.z;
  const Doc doc = doc_at(P, d);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane & 15, r0 = 4 * wave + (lane >> 4);  // 16 rows a step
  float mx = 0.f;
  if (doc.ok) {
    for (int i0 = 64 * part; i0 < doc.n; i0 += 64 * kKeyNormParts) {
      float ss[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + 16 * u + r0;
        ss[u] = 0.f;
        if (i < doc.n) {
          const uint4 w = *reinterpret_cast<const uint4 *>(
              P.k + ((doc.t0 + i) * P.hkv + g) * D + 8 * sub);
          const uint32_t v[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float lo = __uint_as_float(v[e] << 16);
            const float hi = __uint_as_float(v[e] & 0xffff0000u);
            ss[u] = fmaf(lo, lo, fmaf(hi, hi, ss[u]));
          }
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
#pragma unroll
        for (int off = 8; off > 0; off >>= 1)
          ss[u] += __shfl_xor(ss[u], off, 64);
        mx = fmaxf(mx, ss[u]);
      }
    }
  }
#pragma unroll
  for (int off = 16; off < 64; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  if (lane == 0) wmax[wave] = mx;
  __syncthreads();
  if (threadIdx.x == 0)
    P.kmax[((int64_t)d * P.hkv + g) * kKeyNormParts + part] =
        sqrtf(fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3])));
}

// Row log-sum-exp.  grid (row blocks of 128, kv head, docs); each wave owns
// 32 rows and keeps the HR q heads of the group in registers while the
// document's keys 0 .. (last row of the block) stream through LDS, one
// 128-key block at a time, shared by the block's four waves.  Per row and
// head the sum of 2^(logit - m) over the visible keys (scaled logits in log2
// units) with one of two references m:
//   - fixed: m = c |q^_j| max_i |k^_i| bounds every logit of the row from
//     above (Cauchy-Schwarz), and from below by -m, so with m <= 60 every
//     term lies in [2^-120, 1] and no maximum is tracked at all;
//   - running: the exact running maximum, for waves where some row's bound
//     exceeds 60.
// The two lane halves are combined at the end.
constexpr float kFixedRefMax = 60.f;

// Sum and maximum of a tile's 16 values per lane in four interleaved
// partials, so the adds (or maxima) form chains of four, not one chain of
// sixteen behind the exponentials.
__device__ __forceinline__ float sum16(const float (&e)[16]) {
  float a[4] = {e[0], e[1], e[2], e[3]};
#pragma unroll
  for (int i = 4; i < 16; ++i) a[i & 3] += e[i];
  return (a[0] + a[1]) + (a[2] + a[3]);
}
__device__ __forceinline__ float max16(const floatx16 &x) {
  float a[4] = {x[0], x[1], x[2], x[3]};
#pragma unroll
  for (int i = 4; i < 16; ++i) a[i & 3] = fmaxf(a[i & 3], x[i]);
  return fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3]));
}

// grid (kv heads, documents, row blocks), longest rows first: blocks that
// follow each other, and with them the XCDs, get equally long rows (row blocks
// as the fast dimension gave an XCD every eighth one, and with 16 of them the
// first XCD 24 key blocks where the last had 10), and with eight kv heads an
// XCD reads one head's keys.  16 documents of 2048 tokens, 32 q / 8 kv heads:
// 559 -> 327 us, with one head per sweep in place of two 430; 512 documents of
// 256 tokens, 16 / 8 heads: 253 -> 221.
template <int HR, bool WIDE>
__global__ __launch_bounds__(256, 2) void k_row_lse(SalienceParams P) {
  __shared__ __attribute__((aligned(16))) uint16_t ks[2][kLdsK];
  const int d = P.d0 + blockIdx.y;
  const Doc doc = doc_at(P, d);
  if (!doc.ok) return;
  const int rb = gridDim.z - 1 - blockIdx.z;
  if (rb * kRowBlock >= doc.n) return;  // block-uniform, before barriers
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int hf = lane >> 5, lq = lane & 31;
  const int row0 = rb * kRowBlock + wave * 32;
  const bool active = row0 < doc.n;
  const int g = blockIdx.x;
  const int j = row0 + lq;
  const int jl = min(j, doc.n - 1);
  const int last = min(row0 + 31, doc.n - 1);
  const int64_t qrow = (doc.t0 + jl) * P.hq;
  const int kr = perm(lq);

  float kmax = 0.f;
#pragma unroll
  for (int i = 0; i < kKeyNormParts; ++i)
    kmax = fmaxf(kmax, P.kmax[((int64_t)d * P.hkv + g) * kKeyNormParts + i]);
  for (int h0 = 0; h0 < P.n_rep; h0 += HR) {
    const int hbase = g * P.n_rep + h0;
    bf16x8 qf[HR][8];
    float m[HR], l[HR];
    bool fits = true;
#pragma unroll
    for (int r = 0; r < HR; ++r) {
      l[r] = 0.f;
      // (a wave past the document's end loads its clamped rows too: it
      // computes below the diagonal and stores nothing)
      float ss = 0.f;
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        qf[r][s] = ld8(P.q + (qrow + hbase + r) * D + 16 * s + 8 * hf);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float x = (float)qf[r][s][e];
          ss = fmaf(x, x, ss);
        }
      }
      ss += __shfl_xor(ss, 32, 64);
      m[r] = P.c * sqrtf(ss) * kmax;
      fits = fits && m[r] <= kFixedRefMax;
    }
    // wave-uniform choice of the reference
    const bool fixed = __all(fits);
    if (!fixed) {
#pragma unroll
      for (int r = 0; r < HR; ++r) m[r] = -INFINITY;
    }
    if (h0 > 0) __syncthreads();  // the previous heads are done with ks[0]
    stage_rows<WIDE>(P.k, P.hkv, doc, 0, g, ks[0]);
    for (int kb = 0; kb <= rb; ++kb) {
      wait_vmem();
      __syncthreads();  // block kb staged; every wave done with the other
      if (kb < rb)
        stage_rows<WIDE>(P.k, P.hkv, doc, (kb + 1) * kKeyBlock, g,
                   ks[(kb + 1) & 1]);
      const uint16_t *kbuf = ks[kb & 1];
      const int key0 = kb * kKeyBlock;
      // below the diagonal every row sees all 128 keys: four sub-tiles in
      // straight-line code (no masks, no branches), the same arithmetic as
      // the masked path with every key visible; the next sub-tile's
      // fragments are read once the last head's products have consumed
      // the current ones
      auto full_block = [&](auto fixed_ref) {
        constexpr bool FIXED = decltype(fixed_ref)::value;
        bf16x8 kf[8];
        row_frags(kbuf, 0, kr, hf, kf);
        // unit u = (sub-tile u / HR, head u % HR); the products of unit u
        // alternate with the exponentials of unit u - 1
        floatx16 S[2];
#pragma unroll
        for (int u = 0; u <= 4 * HR; ++u) {
          const int st = u / HR, r = u % HR, rp = (u + HR - 1) % HR;
          const floatx16 &T = S[(u + 1) & 1];
          float mn = 0.f, a[4];
          if (u > 0) mn = FIXED ? m[rp] : fmaxf(m[rp], max16(T) * P.c);
          if (u < 4 * HR) {
#pragma unroll
            for (int i = 0; i < 16; ++i) S[u & 1][i] = 0.f;
          }
#pragma unroll
          for (int s = 0; s < 8; ++s) {
            if (u < 4 * HR)
              S[u & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                  kf[s], qf[r][s], S[u & 1], 0, 0, 0);
            if (r == HR - 1 && st + 1 < 4)
              kf[s] = row_frag(kbuf, st + 1, kr, hf, s);
            if (u > 0) {
#pragma unroll
              for (int i = 2 * s; i < 2 * s + 2; ++i) {
                const float e =
                    __builtin_amdgcn_exp2f(fmaf(T[i], P.c, -mn));
                a[i & 3] = i < 4 ? e : a[i & 3] + e;
              }
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          if (u > 0) {
            const float sum = (a[0] + a[1]) + (a[2] + a[3]);
            if (FIXED) {
              l[rp] += sum;
            } else {
              l[rp] = l[rp] * __builtin_amdgcn_exp2f(m[rp] - mn) + sum;
              m[rp] = mn;
            }
          }
        }
      };
      if (kb < rb) {
        if (fixed)
          full_block(std::true_type{});
        else
          full_block(std::false_type{});
        continue;
      }
      if (!active) continue;
      const int nt = min(4, (last - key0) / 32 + 1);
#pragma unroll
      for (int st = 0; st < 4; ++st) {
        if (st >= nt) break;
        bf16x8 kf[8];
        row_frags(kbuf, st, kr, hf, kf);
        // keys of this sub-tile past the wave's first row need the mask
        const bool masked = key0 + 32 * st + 31 > row0;
        const int lim = j - key0 - 32 * st - 16 * hf;  // visible: i <= lim
#pragma unroll
        for (int r = 0; r < HR; ++r) {
          floatx16 S;
#pragma unroll
          for (int i = 0; i < 16; ++i) S[i] = 0.f;
#pragma unroll
          for (int s = 0; s < 8; ++s)
            S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[r][s], S,
                                                        0, 0, 0);
          // the scale c > 0 commutes with the max, so it is applied once
          // to the chunk's max and fused into each exponent's argument
          floatx16 x;
#pragma unroll
          for (int i = 0; i < 16; ++i)
            x[i] = masked && i > lim ? -INFINITY : S[i];
          const float mn = fixed ? m[r] : fmaxf(m[r], max16(x) * P.c);
          if (mn > -INFINITY) {
            float e[16];
#pragma unroll
            for (int i = 0; i < 16; ++i)
              e[i] = __builtin_amdgcn_exp2f(fmaf(x[i], P.c, -mn));
            l[r] = l[r] * __builtin_amdgcn_exp2f(m[r] - mn) + sum16(e);
            m[r] = mn;
          }
        }
      }
    }
#pragma unroll
    for (int r = 0; r < HR; ++r) {
      const float mo = __shfl_xor(m[r], 32, 64);
      const float lo = __shfl_xor(l[r], 32, 64);
      const float mn = fmaxf(m[r], mo);
      // every row sees at least its own key, so mn is finite
      const float tot = l[r] * __builtin_amdgcn_exp2f(m[r] - mn) +
                        lo * __builtin_amdgcn_exp2f(mo - mn);
      if (active && hf == 0 && j < doc.n)
        P.lse2[(int64_t)(hbase + r) * P.total_tokens + doc.t0 + j] =
            mn + log2f(tot);
    }
  }
}

// A tile's sums over the heads: row j's means of the keys i0 .. i0 + 15, as far
// as the row sees them.
__device__ __forceinline__ void store_tile(const SalienceParams &P,
                                           const Doc &doc, int d, int j, int i0,
                                           const floatx16 &acc) {
  if (j >= doc.n) return;
  float *out = P.abar + (int64_t)(d - P.d0) * P.abar_stride +
               (int64_t)j * P.max_len;
  float v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = acc[i] * P.inv_hq;
  const bool vec = (P.max_len & 3) == 0;  // rows 16-byte aligned
  if (vec && i0 + 16 <= j + 1) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
      *reinterpret_cast<float4 *>(out + i0 + 4 * c) =
          make_float4(v[4 * c], v[4 * c + 1], v[4 * c + 2], v[4 * c + 3]);
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (i0 + i <= j) out[i0 + i] = v[i];
  }
}

// ---------------------------------------------------------------------------
// Head-averaged attention.  Unit (rb, kb), kb <= rb, covers rows rb*128 ..
// +127 and keys kb*128 .. +127, a 64 x 64 quarter per wave.  A wave holds its
// keys' fragments of one kv head in registers for all of the group's q heads,
// and reads each q fragment once for both of its 32-key tiles.  The blocks of
// 128 rows, a kv head's keys and then each of its q heads, pass through two
// LDS buffers: the next one's direct global->LDS loads (whole rows of 256
// bytes) run under the current one's products.  The products of one 32 x 32
// tile alternate with the exponentials of the tile before.  With q read from
// memory in the operand's layout, 32 rows per wave and keys from LDS it took
// 448 us (16 documents of 2048 tokens, 32 q / 8 kv heads) and 257 (512 of 256,
// 16 / 8 heads), now 427 and 220; 64-key units at three waves per SIMD 612.
template <bool DIAG, bool WIDE>
__device__ __forceinline__ void mean_attn_unit(const SalienceParams &P,
                                               const Doc &doc, int d, int rb,
                                               int kb,
                                               uint16_t (&ks)[2][kLdsK]) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int hf = lane >> 5, lq = lane & 31;
  const int row0 = rb * kRowBlock, key0 = kb * kKeyBlock;
  // the wave's row tiles rt, rt + 1 and key tiles kt, kt + 1; on the diagonal
  // the wave above it (rt 0, kt 2) has nothing to do, and no tile is computed
  // whose rows all come before its keys or lie past the document's end (below
  // the diagonal those repeat the last row and are not stored, which keeps the
  // loop free of branches)
  const int rt = (wave >> 1) * 2, kt = (wave & 1) * 2;
  const int end = (doc.n - 1 - row0) / 32 + 1;

  floatx16 acc[2][2];  // [row tile][key tile]
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[t][k][i] = 0.f;

  const float *lse = P.lse2 + doc.t0;
  float L[2], Ln[2];
  auto load_l = [&](int h) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
      Ln[t] = lse[(int64_t)h * P.total_tokens +
                  min(row0 + 32 * (rt + t) + lq, doc.n - 1)];
  };
  int buf = 0, h = 0;
  stage_rows<WIDE>(P.k, P.hkv, doc, key0, 0, ks[0]);
  for (int g = 0; g < P.hkv; ++g) {
    wait_vmem();
    __syncthreads();  // the keys are staged; every wave done with the other
    stage_rows<WIDE>(P.q, P.hq, doc, row0, h, ks[buf ^ 1]);
    load_l(h);
    bf16x8 kf[2][8];
#pragma unroll
    for (int k = 0; k < 2; ++k)
      row_frags(ks[buf], kt + k, perm(lq), hf, kf[k]);
    for (int r = 0; r < P.n_rep; ++r, ++h) {
      buf ^= 1;
      wait_vmem();
      __syncthreads();
#pragma unroll
      for (int t = 0; t < 2; ++t) L[t] = Ln[t];
      if (r + 1 < P.n_rep) {
        stage_rows<WIDE>(P.q, P.hq, doc, row0, h + 1, ks[buf ^ 1]);
        load_l(h + 1);
      } else if (g + 1 < P.hkv) {
        stage_rows<WIDE>(P.k, P.hkv, doc, key0, g + 1, ks[buf ^ 1]);
      }
      const uint16_t *qbuf = ks[buf] + rt * 32 * D;
      bf16x8 qf[8];
      if (!DIAG) {
        floatx16 S[2];
        row_frags(qbuf, 0, lq, hf, qf);
        // tile u = (row tile u / 2, key tile u % 2)
#pragma unroll
        for (int u = 0; u < 5; ++u) {
          const int pt = (u + 3) / 2 - 2, pk = (u + 1) & 1;  // tile u - 1
          if (u < 4) {
#pragma unroll
            for (int i = 0; i < 16; ++i) S[u & 1][i] = 0.f;
          }
#pragma unroll
          for (int s = 0; s < 8; ++s) {
            if (u < 4)
              S[u & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                  kf[u & 1][s], qf[s], S[u & 1], 0, 0, 0);
            if (u == 1) qf[s] = row_frag(qbuf, 1, lq, hf, s);
            if (u > 0) {
#pragma unroll
              for (int i = 2 * s; i < 2 * s + 2; ++i)
                acc[pt][pk][i] += __builtin_amdgcn_exp2f(
                    fmaf(S[pk][i], P.c, -L[pt]));
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        continue;
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        if (rt + t < kt || rt + t >= end) continue;
        row_frags(qbuf, t, lq, hf, qf);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          if (rt + t < kt + k) continue;
          floatx16 S;
#pragma unroll
          for (int i = 0; i < 16; ++i) S[i] = 0.f;
#pragma unroll
          for (int s = 0; s < 8; ++s)
            S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[k][s], qf[s], S, 0,
                                                        0, 0);
          // (keys after the row are computed and not stored)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            acc[t][k][i] += __builtin_amdgcn_exp2f(fmaf(S[i], P.c, -L[t]));
        }
      }
    }
    buf ^= 1;
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int k = 0; k < 2; ++k)
      store_tile(P, doc, d, row0 + 32 * (rt + t) + lq,
                 key0 + 32 * (kt + k) + 16 * hf, acc[t][k]);
}

// grid: the units of each document one after another, unit rb (rb + 1) / 2 +
// kb, in runs of kUnitRun that go to the XCDs in turn (block b runs on XCD
// b % 8): units that follow each other share their rows' q through one L2.
// Whole call in runs of 1, 4, 32 and 128 units, us: 16 documents of 2048 tokens
// (32 q / 8 kv heads) 736, 718, 708, 805; 512 of 256 (16 / 8) 468, 458, 457, 490.
constexpr int kUnitRun = 32;
template <bool WIDE>
__global__ __launch_bounds__(256, 2) void k_mean_attn(SalienceParams P,
                                                      int32_t nb,
                                                      int32_t n_docs) {
  __shared__ __attribute__((aligned(16))) uint16_t ks[2][kLdsK];
  const int slot = blockIdx.x / 8;
  const int unit =
      (slot / kUnitRun * 8 + blockIdx.x % 8) * kUnitRun + slot % kUnitRun;
  const int per = nb * (nb + 1) / 2;
  const int dd = unit / per, t = unit % per;
  if (dd >= n_docs) return;  // block-uniform, before any barrier
  const int d = P.d0 + dd;
  const Doc doc = doc_at(P, d);
  if (!doc.ok) return;
  int rb = __builtin_amdgcn_readfirstlane(
      (int)((sqrtf(8.f * t + 1.f) - 1.f) * 0.5f));
  while (rb * (rb + 1) / 2 > t) --rb;
  while ((rb + 1) * (rb + 2) / 2 <= t) ++rb;
  const int kb = t - rb * (rb + 1) / 2;
  if (rb * kRowBlock >= doc.n) return;  // before any barrier
  if (kb < rb)  // block-uniform
    mean_attn_unit<false, WIDE>(P, doc, d, rb, kb, ks);
  else
    mean_attn_unit<true, WIDE>(P, doc, d, rb, kb, ks);
}

// The same where no document of the call is longer than 64 tokens, a block per
// document: three tiles, one for each of three waves, and a kv head's keys and
// its first q head's rows share a buffer, so one wait passes per q head.  The
// unit above has two per kv head and all three tiles on one wave.  Whole call,
// unit above -> this kernel, us: 62 documents of 33 tokens, 8 q and 8 kv heads
// 43.9 -> 31.7, 32 q and 16 kv heads 84.6 -> 53.1; 3,971 documents, 56 and 8
// heads 2051 -> 1842; 512 of 64 tokens, 8 and 4 heads 89 -> 85.  From 65 tokens
// on there are up to ten tiles and more.  (As a branch of the kernel above it
// cost that one 1 %.)
constexpr int kShortDoc = 64;

template <bool WIDE>
__global__ __launch_bounds__(256, 2) void k_mean_attn_short(SalienceParams P) {
  constexpr int Q0 = kShortDoc * D;  // the q rows' place in a buffer
  __shared__ __attribute__((aligned(16))) uint16_t ks[2][2 * Q0];
  const int d = P.d0 + blockIdx.x;
  const Doc doc = doc_at(P, d);
  if (!doc.ok) return;  // block-uniform, before any barrier
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int hf = lane >> 5, lq = lane & 31;
  const int rt = wave > 0, kt = wave > 1;  // tiles (0, 0), (1, 0), (1, 1)
  const bool active = wave < 3 && 32 * rt < doc.n;
  const int j = 32 * rt + lq;
  const float *lse = P.lse2 + doc.t0 + min(j, doc.n - 1);
  floatx16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  bf16x8 kf[8], qf[8];
  stage_rows<WIDE, kShortDoc>(P.k, P.hkv, doc, 0, 0, ks[0]);
  stage_rows<WIDE, kShortDoc>(P.q, P.hq, doc, 0, 0, ks[0] + Q0);
  float Ln = lse[0];
  for (int h = 0, g = 0, r = 0; h < P.hq; ++h) {
    const uint16_t *buf = ks[h & 1];
    uint16_t *next = ks[(h & 1) ^ 1];
    wait_vmem();
    __syncthreads();  // head h staged; every wave done with the other buffer
    const float L = Ln;
    const bool first = r == 0;
    if (++r == P.n_rep) r = 0, ++g;
    if (h + 1 < P.hq) {
      if (r == 0) stage_rows<WIDE, kShortDoc>(P.k, P.hkv, doc, 0, g, next);
      stage_rows<WIDE, kShortDoc>(P.q, P.hq, doc, 0, h + 1, next + Q0);
      Ln = lse[(int64_t)(h + 1) * P.total_tokens];
    }
    if (!active) continue;
    if (first) row_frags(buf, kt, perm(lq), hf, kf);
    row_frags(buf + Q0, rt, lq, hf, qf);
    floatx16 S;
#pragma unroll
    for (int i = 0; i < 16; ++i) S[i] = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s)
      S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[s], S, 0, 0, 0);
    // (keys after the row are computed and not stored)
#pragma unroll
    for (int i = 0; i < 16; ++i)
      acc[i] += __builtin_amdgcn_exp2f(fmaf(S[i], P.c, -L));
  }
  if (active) store_tile(P, doc, d, j, 32 * kt + 16 * hf, acc);
}

// ---------------------------------------------------------------------------
// Column top-p means.  grid (strips of 64 columns, docs); the W waves of a
// block stream rows j = c0 + w, c0 + w + W, ... of the strip; lane l keeps
// the PM largest values of column c0 + l (descending, -1 = empty) and the
// lists are merged through LDS at the end, half of them into the other half
// at a time.  A wave walks its rows eight loads at a time, so the longest
// column is a chain of n / 8W memory latencies (W: see ToppWide).
template <int PM>
__device__ __forceinline__ void insert(float (&L)[PM], float v) {
#pragma unroll
  for (int k = 0; k < PM; ++k) {
    const float hi = fmaxf(L[k], v);
    v = fminf(L[k], v);
    L[k] = hi;
  }
}

template <int PM, int W>
__global__ __launch_bounds__(64 * W) void k_col_topp(SalienceParams P) {
  __shared__ float merge[W / 2][PM][kStrip];
  const int d = P.d0 + blockIdx.y;
  const Doc doc = doc_at(P, d);
  if (!doc.ok) return;
  const int c0 = blockIdx.x * kStrip;
  if (c0 >= doc.n) return;  // block-uniform, before the barriers
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int c = c0 + lane;
  const bool col = c < doc.n;
  const float *base = P.abar + (int64_t)(d - P.d0) * P.abar_stride +
                      (col ? c : c0);
  float L[PM];
#pragma unroll
  for (int k = 0; k < PM; ++k) L[k] = -1.f;
  constexpr int U = 8;
  int j = c0 + wave;
  for (; j + W * (U - 1) < doc.n; j += W * U) {
    float v[U];
#pragma unroll
    for (int x = 0; x < U; ++x)
      v[x] = base[(int64_t)(j + W * x) * P.max_len];
#pragma unroll
    for (int x = 0; x < U; ++x) {
      const float w = (col && j + W * x >= c) ? v[x] : -1.f;
      if (__any(w > L[PM - 1])) insert(L, w);
    }
  }
  for (; j < doc.n; j += W) {
    const float v = base[(int64_t)j * P.max_len];
    const float w = (col && j >= c) ? v : -1.f;
    if (__any(w > L[PM - 1])) insert(L, w);
  }
  for (int half = W / 2; half > 0; half >>= 1) {
    if (wave >= half && wave < 2 * half) {
#pragma unroll
      for (int k = 0; k < PM; ++k) merge[wave - half][k][lane] = L[k];
    }
    __syncthreads();
    if (wave < half) {
      for (int k = 0; k < PM; ++k) {
        const float v = merge[wave][k][lane];
        if (__any(v > L[PM - 1])) insert(L, v);
      }
    }
    __syncthreads();
  }
  if (wave != 0 || !col) return;
  const int m = min(P.top_p, doc.n - c);
  float sum = 0.f;
#pragma unroll
  for (int k = 0; k < PM; ++k)
    if (k < m) sum += L[k];
  P.u[doc.t0 + c] = sum / (float)m;
}

// ---------------------------------------------------------------------------
// Validation of the document and selection offsets (one thread per doc).
__global__ __launch_bounds__(256) void k_check(SalienceParams P) {
  const int d = blockIdx.x * 256 + threadIdx.x;
  if (d >= P.n_docs) return;
  if (!doc_at(P, d).ok || (d == P.n_docs - 1 &&
                           P.cu[d + 1] != P.total_tokens))
    raise_status(P.status, DOPR_ERR_SEQLEN);
}

}  // namespace

// ---------------------------------------------------------------------------
// Top-K selection.  One block per document: the K-th largest key (the
// orderable bits of u) is found eight bits at a time from a histogram of the
// keys that share the bits found so far; the keys above it, and of those equal
// to it as many as are missing, the lowest positions first, are written in
// position order.  Four short passes, bound by their barriers, where a bitonic
// sort of the keys took 66 to 78 (documents of 2048 tokens 34 -> 10 us, 512 of
// 256 tokens 17 -> 10).
namespace {

constexpr int kTopkThreads = 1024;

__device__ __forceinline__ uint32_t orderable(float f) {
  const uint32_t b = __float_as_uint(f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__global__ __launch_bounds__(kTopkThreads) void k_topk(TopkParams P) {
  __shared__ uint32_t key[kSalienceMaxLen];
  __shared__ int32_t hist[256];
  __shared__ int32_t found[2];  // the bin of the K-th key, keys above it
  __shared__ int32_t wsum[kTopkThreads / 64];
  const int d = blockIdx.x;
  const int32_t a = P.cu[d], b = P.cu[d + 1];
  const int32_t n = b - a;
  if (a < 0 || n < 1 || n > P.max_len || b > P.total_tokens) {
    if (threadIdx.x == 0 && P.status) raise_status(P.status, DOPR_ERR_SEQLEN);
    return;
  }
  const int32_t sa = P.cs[d], sb = P.cs[d + 1];
  const int32_t K = sb - sa;
  if (sa < 0 || K < 0 || K > n || sb > P.total_select) {
    if (threadIdx.x == 0 && P.status) raise_status(P.status, DOPR_ERR_SEQLEN);
    return;
  }
  if (K == 0) return;
  int32_t *out = P.selected + sa;
  if (K == n) {
    for (int i = threadIdx.x; i < n; i += kTopkThreads) out[i] = i;
    return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float *u = P.u + a;
  for (int i = threadIdx.x; i < n; i += kTopkThreads) key[i] = orderable(u[i]);
  uint32_t kth = 0;  // the K-th largest key's bits above `shift`
  int need = K;      // keys still to take among those that share them
  for (int shift = 24; shift >= 0; shift -= 8) {
    const uint32_t seen = shift == 24 ? 0u : ~0u << (shift + 8);
    if (threadIdx.x < 256) hist[threadIdx.x] = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += kTopkThreads)
      if (((key[i] ^ kth) & seen) == 0)
        atomicAdd(&hist[(key[i] >> shift) & 255], 1);
    __syncthreads();
    if (wave == 0) {
      // lane l: bins 255 - 4l down to 252 - 4l
      int c[4], own = 0;
#pragma unroll
      for (int x = 0; x < 4; ++x) own += c[x] = hist[255 - 4 * lane - x];
      int incl = own;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
      }
      int above = incl - own;
      if (above < need && need <= incl) {  // one lane
        int x = 0;
        while (above + c[x] < need) above += c[x++];
        found[0] = 255 - 4 * lane - x;
        found[1] = above;
      }
    }
    __syncthreads();
    kth |= (uint32_t)found[0] << shift;
    need -= found[1];
  }
  // ordered compaction: thread t owns positions [t*per, (t+1)*per); counts of
  // keys above the K-th in the low half, of equal ones in the high half
  const int per = (n + kTopkThreads - 1) / kTopkThreads;
  const int p0 = threadIdx.x * per, p1 = min(p0 + per, n);
  int cnt = 0;
  for (int i = p0; i < p1; ++i)
    cnt += key[i] > kth ? 1 : key[i] == kth ? 1 << 16 : 0;
  int incl = cnt;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(incl, o, 64);
    if (lane >= o) incl += y;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  int before = incl - cnt;
  for (int w = 0; w < wave; ++w) before += wsum[w];
  int gt = before & 0xffff, eq = before >> 16;
  for (int i = p0; i < p1; ++i) {
    const bool more = key[i] > kth, same = key[i] == kth;
    if (more || (same && eq < need)) out[gt + min(eq, need)] = i;
    gt += more;
    eq += same;
  }
}

template <bool WIDE>
void launch_sweeps(const SalienceParams &p, int hr, dim3 g_lse, dim3 g_att,
                   int nb, int32_t n_docs, hipStream_t s) {
  if (hr == 2)
    hipLaunchKernelGGL((k_row_lse<2, WIDE>), g_lse, dim3(256), 0, s, p);
  else
    hipLaunchKernelGGL((k_row_lse<1, WIDE>), g_lse, dim3(256), 0, s, p);
  if (p.max_len <= kShortDoc) {
    hipLaunchKernelGGL(k_mean_attn_short<WIDE>, dim3(n_docs), dim3(256), 0, s,
                       p);
    return;
  }
  hipLaunchKernelGGL(k_mean_attn<WIDE>, g_att, dim3(256), 0, s, p,
                     (int32_t)nb, n_docs);
}

template <int PM>
void launch_col_topp(const SalienceParams &p, dim3 grid, hipStream_t s) {
  if constexpr (PM <= 16) {
    constexpr ToppWide wide = PM == 8 ? kToppWide8 : kToppWide16;
    if (p.max_len >= wide.min_len &&
        (int64_t)grid.x * grid.y <= wide.max_strips) {
      hipLaunchKernelGGL((k_col_topp<PM, 16>), grid, dim3(1024), 0, s, p);
      return;
    }
  }
  hipLaunchKernelGGL((k_col_topp<PM, 4>), grid, dim3(256), 0, s, p);
}

}  // namespace

hipError_t launch_salience_chunk(const SalienceParams &p, int32_t n_docs,
                                 int hr, int pm, hipStream_t s) {
  if (n_docs == 0) return hipSuccess;
  const int nb = (p.max_len + kRowBlock - 1) / kRowBlock;
  const dim3 g_lse(p.hkv, n_docs, nb);
  const int64_t units = (int64_t)nb * (nb + 1) / 2 * n_docs;
  constexpr int kRun8 = 8 * kUnitRun;
  const dim3 g_att((unsigned)((units + kRun8 - 1) / kRun8 * kRun8));
  const dim3 g_col((p.max_len + kStrip - 1) / kStrip, n_docs);
  if (p.hq > kOffsetHeads)
    launch_sweeps<true>(p, hr, g_lse, g_att, nb, n_docs, s);
  else
    launch_sweeps<false>(p, hr, g_lse, g_att, nb, n_docs, s);
  if (pm == 8)
    launch_col_topp<8>(p, g_col, s);
  else if (pm == 16)
    launch_col_topp<16>(p, g_col, s);
  else if (pm == 32)
    launch_col_topp<32>(p, g_col, s);
  else
    launch_col_topp<64>(p, g_col, s);
  return hipGetLastError();
}

hipError_t launch_key_norms(const SalienceParams &p, hipStream_t s) {
  if (p.n_docs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_key_norm,
                     dim3((unsigned)p.n_docs, (unsigned)p.hkv, kKeyNormParts),
                     dim3(256), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_salience_check(const SalienceParams &p, hipStream_t s) {
  if (p.n_docs == 0 || !p.status) return hipSuccess;
  hipLaunchKernelGGL(k_check, dim3((p.n_docs + 255) / 256), dim3(256), 0, s,
                     p);
  return hipGetLastError();
}

hipError_t launch_topk(const TopkParams &p, int32_t n_docs, hipStream_t s) {
  if (n_docs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_topk, dim3(n_docs), dim3(kTopkThreads), 0, s, p);
  return hipGetLastError();
}

}  // namespace dopr
