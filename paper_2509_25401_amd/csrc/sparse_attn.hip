// FlashOmni attention (Algorithm 1 of the paper) for AMD MI355X / gfx950.
//
// Two kernels per call, both on the caller's stream (the second alone where the order of the rows does not matter, few
// rows, or no symbols and at most two rows per workgroup, and where its workgroups sort the rows themselves, a few rows per CU;
// one more, decode_rows, where a queue has many symbols):
//   plan_queues decodes the packed symbols of Section 3.3 once per (b,h,i) row into aligned
//               32-bit words (bit j of the row = key block j, padding cleared), counts the
//               kept key blocks of every non-cached row and notes the first of them;
//               sorts the rows into one work queue per XCD (a head's rows all go to one XCD, so
//               its K/V stream through one L2): rows that are a large part of a workgroup's
//               share first (longest first), the others head by head and heaviest first inside a
//               head (55 kept-count buckets), cached rows (plain copies) last;
//   attn        a persistent grid that fills the CUs (two workgroups of 128 query rows each, three with 64 channels) pulls items
//               from its XCD's queue and steals from the others when that is drained.  A compute item is one query block:
//               Q lives in registers as stored (the 1/sqrt(D) scale is applied to the fp32 score),
//               the reduction-axis symbol is walked with scalar find-first-set on the decoded words, and only kept
//               K/V tiles are streamed to LDS with direct-to-LDS loads, double buffered in 64-key
//               sub-tiles.  S^T = K Q^T and O^T = V^T P^T run on v_mfma_f32_32x32x16_bf16, so
//               each lane owns one query row: the row maximum needs a single half-wave exchange,
//               the row sum none until the end, and the exponentiated S^T accumulators are the
//               B operand of the O^T product without any data movement.  The reference of the
//               exponent is the C operand of the first S^T MFMA; it is checked after the fact
//               (the sum of a block's weights shows whether a score left the allowed range)
//               and moves only then, so the steady state takes no row maximum at all.  The
//               vector instructions of the softmax sit between matrix instructions that do not
//               depend on them (weights of one 32-key block under the scores of the next and
//               under the O^T product of the previous), where they issue in the shadow of the
//               wave's own MFMAs.  The finished block leaves through LDS as whole rows.  The ticket
//               of the next item is drawn a few key blocks before the current one ends, and its
//               work-list entry names the first kept key block, so that tile is requested before
//               the row's symbol words are touched.  A copy item moves one cached block
//               O_cache -> O.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <map>
#include <mutex>
#include <new>
#include <type_traits>
#include <utility>

#include "sparse_attn.h"
#include "sparse_attn_internal.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;

// f(integral_constant 0), ..., f(integral_constant N - 1)
template <int... I, typename F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, const F& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(const F& f) {
  static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

#define LDS_PTR(T) T __attribute__((address_space(3)))*
#define GLOBAL_PTR(T) T __attribute__((address_space(1)))*

// Keys per LDS sub-tile: 64, except for 64-row blocks of 128 channels when there are many of them.  Four K and V sub-tiles
// of 64 keys are 64 KiB, of which a CU holds two, and two workgroups of two waves leave half of its waves idle; with 32
// keys it holds four (24 heads, us, 64 / 32 keys: 9001 tokens at 40 % keep 655 / 478, 33024 tokens at 25 % keep and 50 % cached
// 2276 / 1834).  A workgroup by itself is quicker with 64, where the softmax of one half lies under the matrix
// instructions of the other, so 64 as long as a CU has no more than about two rows to compute: up to two rows per CU, or
// three where some are cached (24 heads, 30 % keep: 1344 tokens, 504 rows, 20.4 / 20.8 and half of them cached 19.6 / 21.3;
// 2048 tokens, 768 rows, none cached 37 / 30, half of them cached 27.6 / 32.7).  A mask whose time is that of a few heavy
// rows among many light ones loses with 32 as well (9001 tokens, 2 % of the rows at 95 %, the others at 3 %: 213 / 240); that
// is not known when the kernel is chosen.
constexpr int attn_keys(int D, int bq, long long rows, bool some_cached, int cus) {
  return D == 128 && bq == 64 && rows > (some_cached ? 3LL : 2LL) * cus ? 32 : 64;
}
// How the rows (query blocks) get to the workgroups.
//   kQueues  plan_queues has ordered them; tickets, stealing
//   kDealt   by workgroup number, every workgroup decodes the symbols of its rows: where the order does not matter
//   kSorted  every workgroup decodes and sorts the rows of its XCD (an eighth of all, at most kSortRows of kSortWords words) and
//            takes those that fall to its number, the longest first; cached rows go to workgroups without a computed one.  For
//            calls of a few rows per CU, where the pre-pass is a large part of the time (see run())
enum : int { kQueues = 0, kDealt = 1, kSorted = 2 };
constexpr int kSortRows = 256, kSortWords = 4;
constexpr int kSortLds = kSortRows * 4 * 2 + kSortRows * kSortWords * 4 + 16;   // keys, list, words, number of computed rows

// Wavefronts per SIMD that the registers are laid out for.  64 channels leave room for three (168 registers, no spill), which
// 128-row blocks use (three workgroups of 32 KiB LDS per CU; 24 heads, us, two / three: 9001 tokens dense 577 / 552, 33024
// tokens at 25 % keep 1745 / 1681; sorted calls, 4608 tokens, 90 % keep 148 / 135, 30 % 53 / 48; 8 heads of 12544 tokens, 90 % keep,
// 388 / 345; 24 calls of 97 to 141 rows per XCD: none slower); of the 64-row workgroups LDS holds four, two wavefronts per SIMD,
// either way.  Dealt instances take up to 172 registers and would spill.
constexpr int attn_waves_per_simd(int D, int mode) { return D == 64 && mode != kDealt ? 3 : 2; }
constexpr int kLongBuckets = 8;       // kept-count buckets of the long rows of a queue (longest first, across heads)
constexpr int kFineBuckets = 55;      // ... of its other rows (head by head); with the bucket of cached rows: 64,
constexpr int kCachedBucket = kLongBuckets + kFineBuckets;   // one lane each in the ranking pass
// Workgroups per XCD that the ordering plans for: those of 128-row blocks (32 CUs x 2).  64-row blocks have twice as many;
// for them a long row is one of two thirds of a share instead of one third, which is the better line for nearly equal
// rows and the worse one for some skewed masks (24 heads, 9001 tokens, 64 x 128 blocks, us, line at two thirds / one
// third: the ragged mask at 40 % keep 225 / 235, a tenth of the rows at 90 % and the others at 10 % 164 / 169, a fifth at 50 % and
// the others at 10 % 166 / 143).  128-row blocks of 64 channels run 96, and are not better off with a line for these (64 / 96: 9001
// tokens, 40 % keep, 25 % cached 198 / 196, 7500 tokens, 90 % keep 359 / 369, 16000 tokens 367 / 371, 33024 tokens 1649 / 1648).
constexpr int kWgsPerXcd = 64;
constexpr int kCusPerXcd = 32;
constexpr int kXcds = 8;               // accelerator dies (XCDs) of the MI355X, each with its own L2
constexpr int kMaxHeadGroups = 24;    // head groups per bucket in the ordering histogram of a queue (6 KiB of LDS)
constexpr int kMaxTq = 16384;
constexpr unsigned kCopyFlag = 0x80000000u;
// Queue counters: every queue head (items handed out so far) sits in a 128-byte line of its own: all workgroups of an
// XCD bump the same head once per item; eight heads in one line would make every workgroup of the chip contend for
// that line.  Behind them the number of workgroups that are done (stored plans).
constexpr int kHeadStride = 32;                   // words between two queue heads
constexpr int kDoneOffset = 8 * kHeadStride;
constexpr int kQueueWords = kDoneOffset + 64;     // 1280 bytes
constexpr int kHwRegXccId = (3 << 11) | 20;   // s_getreg operand: 4 bits at offset 0 of hardware register 20 (XCC_ID)
constexpr int kOrderThreads = 1024;
constexpr int kMaxTerms = 4;            // stored feature + up to three derivatives
constexpr int kMfmaPrio = 1;            // wave priority while it feeds the matrix pipe
constexpr float kSumLimit = 256.0f;     // a lane's 16 weights of one 32-key block may add up to this before the reference moves

struct AttnParams {
  const char* Q;
  const char* K;
  const char* V;
  const char* O_cache;
  char* O;
  const uint32_t* words;   // [N][nw32] decoded symbol words
  const uint32_t* order;   // [N][2] work list: {row | kCopyFlag, sort key of the row (see plan_queues)}
  uint32_t* queues;        // kXcds queue heads at [q * kHeadStride]; (kQueues)
  int mode;                // kQueues ..
  int self_reset;          // the last workgroup to finish clears the queue heads for the next run
  const uint8_t* raw_flags;   // symbols as the caller gave them, nullptr: none (read where items are dealt out)
  const uint8_t* raw_mask;
  int raw_row_bytes;
  int N;                   // B*H*Tq
  int BH;
  int Tq;
  int Tkv;
  int L;
  int nw32;
  int do_copy;             // 0: cached blocks are already in place
  float scale_log2;        // log2(e) / sqrt(D)
  // OP_reuse as a Taylor forecast: cached block = sum_d coef[d] * term[d]; term[0] is O_cache.
  // n_terms == 0 selects the plain bit-exact copy.
  const char* term[kMaxTerms - 1];
  float coef[kMaxTerms];
  int n_terms;
};

// ---------------------------------------------------------------------------------------
// Symbol pre-pass
// ---------------------------------------------------------------------------------------
// Rows and queues.  Head bh belongs to queue (XCD) bh % kXcds; the work list holds the queues one behind the other, so
// where a queue begins follows from the shape.
__host__ __device__ inline int queue_first_head(int q, int BH) { return q * (BH / kXcds) + (q < BH % kXcds ? q : BH % kXcds); }

// One decoded word of a symbol row given as bytes: bit j = key block 32 * w + j, padding cleared.
__device__ inline uint32_t clear_padding(uint32_t word, int w, int Tkv) {
  const int valid = Tkv - 32 * w;   // >= 1 by construction of nw32
  return valid < 32 ? word & ((1u << valid) - 1u) : word;
}

// Work list order: one queue per XCD (head bh belongs to XCD bh % kXcds), in three parts.
//   long rows    rows with more kept blocks than `limit` = a third of what one workgroup gets to do in total
//                (kept blocks of the queue / (3 * kWgsPerXcd); see there for 64-row blocks): longest first across heads (kLongBuckets buckets,
//                heads adjacent inside a bucket), so that none of them starts late.  Uniform masks have none; with
//                few rows per workgroup (short sequences) every row is long.
//   other rows   head by head, inside a head the heaviest first (kFineBuckets buckets), inside a bucket in sequence
//                order.  All workgroups of an XCD then stream the K/V of the same head at the same time, and because
//                rows that run at the same time have (almost) the same number of kept blocks they also stay at
//                about the same key position while they sweep it: a tile one of them has fetched is still in that
//                XCD's L2 when the others ask for it.  What counts for the balance is the end of the queue, and
//                there the light rows of the last head come last.
//   cached rows  (plain copies) of all heads at the very end.
// Bucket of a row: 0 .. kLongBuckets-1 long (heaviest = 0), then kFineBuckets buckets, then kCachedBucket.
// `lightest` = the smallest kept count among the queue's computed rows: the fine buckets span lightest .. limit, so
// that masks whose rows differ by a few blocks only are still sorted block by block.
// The long buckets likewise span the counts that long rows really have (long_lo + 1 .. heaviest).
struct OrderScale {
  int limit, long_lo, heaviest, lightest;
};
__device__ inline int order_major(int key, const OrderScale& sc) {
  if (key < 0) return kCachedBucket;
  const int count = key & 0xffff;   // < 2^16, bucket counts < 2^6: the products fit in 32 bits
  if (count > sc.limit)
    return (kLongBuckets - 1) - (int)((unsigned)(count - sc.long_lo - 1) * kLongBuckets / (unsigned)(sc.heaviest - sc.long_lo));
  return kLongBuckets + (kFineBuckets - 1) -
         (int)((unsigned)(count - sc.lightest) * kFineBuckets / (unsigned)(sc.limit - sc.lightest + 1));
}

// Word w of a row at granularity gran > 1: tile j reads bit j / gran.
__device__ inline uint32_t granular_word(const uint8_t* src, int w, int Tkv, int gran) {
  uint32_t word = 0;
  for (int t = 0; t < 32 && 32 * w + t < Tkv; ++t) {
    const int js = (32 * w + t) / gran;
    word |= (uint32_t)((src[js >> 3] >> (7 - (js & 7))) & 1) << t;
  }
  return word;
}
// Key of a row: kept blocks in the low 16 bits (0 .. 32768), first kept block above them; -1 for cached rows.
__device__ inline int row_key(bool cached, int count, int first_kept) { return cached ? -1 : (count | (max(first_kept, 0) << 16)); }

// Decodes the rows of all queues, 16 lanes to a row: words and keys for plan_queues, which does it by itself where there
// are few words (see launch_plan).
__global__ void __launch_bounds__(256) decode_rows(const uint8_t* __restrict__ cache_flags, const uint8_t* __restrict__ kv_mask,
                                                   int N, int Tq, int Tkv, int gran, int sym_Tq, int sym_row_bytes, int nw32,
                                                   uint32_t* __restrict__ words, int32_t* __restrict__ keys) {
  const int row = (int)blockIdx.x * 16 + (int)threadIdx.x / 16, l16 = threadIdx.x % 16;
  if (row >= N) return;                            // (16 lanes at a time)
  const int bh = row / Tq;
  const size_t sym_row = (size_t)bh * sym_Tq + (row - bh * Tq) / gran;
  const bool cached = cache_flags != nullptr && cache_flags[sym_row] != 0;
  const uint8_t* src = kv_mask ? kv_mask + sym_row * sym_row_bytes : nullptr;
  int count = 0, first_kept = 0x7fffffff;
  for (int w = l16; w < nw32; w += 16) {
    uint32_t word = cached ? 0u : 0xffffffffu;
    if (!cached && src) {
      if (gran == 1) {
        word = 0;
        for (int b = 0; b < 4; ++b) {
          const int byte = 4 * w + b;
          if (byte < sym_row_bytes) word |= (uint32_t)src[byte] << (8 * b);
        }
        word = __builtin_bswap32(__brev(word));    // most significant bit first inside each byte
      } else {
        word = granular_word(src, w, Tkv, gran);
      }
    }
    word = clear_padding(word, w, Tkv);
    words[(size_t)row * nw32 + w] = word;
    count += __popc(word);
    if (word != 0u) first_kept = min(first_kept, 32 * w + __ffs(word) - 1);
  }
  for (int off = 8; off > 0; off >>= 1) {
    count += __shfl_xor(count, off);
    first_kept = min(first_kept, __shfl_xor(first_kept, off));
  }
  if (l16 == 0) keys[row] = row_key(cached, count, count > 0 ? first_kept : 0);
}

// Symbol pre-pass: workgroup q decodes the rows of queue q (unless decode_rows has done so) and writes its part of the
// work list.
//   decode     one thread per row turns the packed symbols into aligned words, counts the kept key blocks and notes
//              the first of them (key of the row; -1 for cached rows)
//   order      counting sort into the buckets above
// One kernel of eight workgroups, because the queues do not depend on each other; it is a chain of memory and LDS round
// trips.  24 heads: 13 us at 33024 tokens, 7 us at 4608, where a decoding kernel and a single-workgroup sort over all
// queues took 7 + 21 and 5 + 9 us and a launch more.
constexpr int kLdsKeys = 8192;     // rows of a queue whose keys stay in LDS
__global__ void __launch_bounds__(kOrderThreads) plan_queues(const uint8_t* __restrict__ cache_flags,
                                                             const uint8_t* __restrict__ kv_mask, int BH, int Tq, int Tkv,
                                                             int gran, int sym_Tq, int sym_row_bytes, int nw32, int shift,
                                                             int groups, bool decoded, uint32_t* __restrict__ words, int32_t* keys,
                                                             uint32_t* __restrict__ order, uint32_t* __restrict__ queues) {
  __shared__ uint32_t bins[(kCachedBucket + 1) * kMaxHeadGroups];
  __shared__ int32_t lds_keys[kLdsKeys];
  __shared__ uint32_t wave_part[kOrderThreads / 64];
  __shared__ unsigned long long kept_all;            // kept key blocks of all rows of the queue
  __shared__ uint32_t heaviest, lightest_u;          // largest / smallest kept count of its computed rows
  __shared__ uint32_t seen_rows[kOrderThreads / 64][64];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int q = blockIdx.x;
  const int heads = (BH - q + kXcds - 1) / kXcds;    // bh = q, q + 8, ...
  const int rows = heads * Tq;                       // local row r: head q + 8 * (r / Tq), query block r % Tq
  const int nbins = (kCachedBucket + 1) * groups;
  if (tid == 0) {
    kept_all = 0ull;
    heaviest = 0u;
    lightest_u = 0xffffu;
    queues[q * kHeadStride] = 0u;
    if (q == 0) queues[kDoneOffset] = 0u;
  }
  for (int b = tid; b < nbins; b += kOrderThreads) bins[b] = 0;
  __syncthreads();
  const bool in_lds = rows <= kLdsKeys;
  auto global_row = [&](int r) -> int { return (q + kXcds * (r / Tq)) * Tq + r % Tq; };
  auto key_of = [&](int r) -> int { return in_lds ? lds_keys[r] : keys[global_row(r)]; };

  {
    unsigned long long sum = 0;
    uint32_t hi = 0, lo = 0xffffu;
    for (int r = tid; r < rows; r += kOrderThreads) {
      const int row = global_row(r);
      int key;
      if (decoded) {
        key = keys[row];
      } else {
        // one symbol covers gran x gran tiles: tile (i, j) reads flag i / gran and mask bit (i / gran, j / gran)
        const size_t sym_row = (size_t)(q + kXcds * (r / Tq)) * sym_Tq + (r % Tq) / gran;
        const bool cached = cache_flags != nullptr && cache_flags[sym_row] != 0;
        int count = 0, first_kept = -1;
        auto take = [&](int w, uint32_t word) {
          word = clear_padding(word, w, Tkv);
          words[(size_t)row * nw32 + w] = word;
          count += __popc(word);
          if (first_kept < 0 && word != 0u) first_kept = 32 * w + __ffs(word) - 1;
        };
        const uint8_t* src = kv_mask ? kv_mask + sym_row * sym_row_bytes : nullptr;
        if (cached || !src) {
          for (int w = 0; w < nw32; ++w) take(w, cached ? 0u : 0xffffffffu);
        } else if (gran == 1) {
          // rows start at any byte: aligned words, shifted together; only words that hold a byte of the row are read
          const int skew = (int)((uintptr_t)src & 3);
          const uint32_t* aligned = (const uint32_t*)(src - skew);
          const int last = (skew + sym_row_bytes - 1) / 4;
          for (int w0 = 0; w0 < nw32; w0 += 8) {
            uint32_t d[9];
#pragma unroll
            for (int t = 0; t < 9; ++t) d[t] = w0 + t <= last ? aligned[w0 + t] : 0u;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
              if (w0 + t < nw32) {
                const uint32_t v = (uint32_t)(((unsigned long long)d[t + 1] << 32 | d[t]) >> (8 * skew));
                take(w0 + t, __builtin_bswap32(__brev(v)));      // most significant bit first inside each byte
              }
            }
          }
        } else {
          for (int w = 0; w < nw32; ++w) take(w, granular_word(src, w, Tkv, gran));
        }
        key = row_key(cached, count, first_kept);
      }
      if (in_lds)
        lds_keys[r] = key;
      else if (!decoded)
        keys[row] = key;
      if (key >= 0) {
        const uint32_t count = (uint32_t)(key & 0xffff);
        sum += count;
        hi = max(hi, count);
        lo = min(lo, count);
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      sum += __shfl_xor(sum, off);
      hi = max(hi, __shfl_xor(hi, off));
      lo = min(lo, __shfl_xor(lo, off));
    }
    if (lane == 0) {
      atomicAdd(&kept_all, sum);
      atomicMax(&heaviest, hi);
      atomicMin(&lightest_u, lo);
    }
  }
  __syncthreads();                                   // keys and sums are in place
  // long = more than a third of a workgroup's share; where no row is that long the fine buckets end at the heaviest
  // row instead
  const int share = (int)min(kept_all / (3ull * kWgsPerXcd), (unsigned long long)Tkv);
  const int limit = (int)heaviest <= share ? (int)heaviest : share;
  const OrderScale sc = {limit, max(limit, (int)min(lightest_u, heaviest) - 1), (int)heaviest, min((int)lightest_u, limit)};
  auto bin_of = [&](int major, int head) -> int {     // head: of this queue, 0 ..
    const int group = head >> shift;
    if (major < kLongBuckets) return major * groups + group;
    if (major < kCachedBucket) return kLongBuckets * groups + group * kFineBuckets + (major - kLongBuckets);
    return kCachedBucket * groups + group;
  };
  for (int r = tid; r < rows; r += kOrderThreads) atomicAdd(&bins[bin_of(order_major(key_of(r), sc), r / Tq)], 1u);
  __syncthreads();
  // exclusive scan of the bins: a contiguous chunk per thread, then over the lanes of a wave, then over the waves
  {
    const int chunk = (nbins + kOrderThreads - 1) / kOrderThreads;
    const int lo = min(nbins, tid * chunk), hi = min(nbins, lo + chunk);
    uint32_t sum = 0;
    for (int b = lo; b < hi; ++b) sum += bins[b];
    uint32_t scan = sum;
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t add = __shfl_up(scan, off);
      scan += lane >= off ? add : 0u;
    }
    if (lane == 63) wave_part[wave] = scan;
    __syncthreads();
    uint32_t run = scan - sum;
    for (int w = 0; w < wave; ++w) run += wave_part[w];
    for (int b = lo; b < hi; ++b) {
      const uint32_t c = bins[b];
      bins[b] = run;
      run += c;
    }
  }
  __syncthreads();
  uint32_t* const list = order + 2 * (size_t)Tq * queue_first_head(q, BH);
  // Inside a bin the rows keep their order in the sequence: neighbouring query blocks, which with windowed symbols
  // keep nearly the same key blocks, are then worked on at the same time and find each other's tiles in L2.  A bin
  // holds rows of one head as long as there are no more than kMaxHeadGroups heads per queue: a wave then walks a
  // head 64 query blocks at a time, keeps the number of rows seen so far in every bucket, and a row's place is the
  // start of its bin + that count + the rows of its bucket at lower lanes (ballots).  With more heads several of them
  // share a bin and the rows take their places in arrival order.
  if (shift == 0) {
    volatile uint32_t* seen = seen_rows[wave];   // rows of the current head met so far, per bucket
    for (int hl = wave; hl < heads; hl += kOrderThreads / 64) {
      seen[lane] = 0u;
      for (int i0 = 0; i0 < Tq; i0 += 64) {
        const bool valid = i0 + lane < Tq;
        const int i = min(i0 + lane, Tq - 1);
        const int key = in_lds ? lds_keys[hl * Tq + i] : keys[(q + kXcds * hl) * Tq + i];
        const int major = valid ? order_major(key, sc) : 0;
        // the lanes whose row falls into the same bucket as this lane's: one ballot per bit of the bucket number
        unsigned long long same = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 6; ++b) {
          const unsigned long long set = __ballot((major >> b) & 1);
          same &= ((major >> b) & 1) ? set : ~set;
        }
        if (valid) {
          // LDS accesses of a wave execute in program order: every lane reads its bucket's count before the first
          // lane of each bucket moves it on
          const uint32_t before = seen[major];
          const uint32_t rank = before + (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
          if ((same & ((1ull << lane) - 1ull)) == 0ull) seen[major] = before + (uint32_t)__popcll(same);
          const uint32_t pos = bins[bin_of(major, hl)] + rank;
          list[2 * pos] = (uint32_t)((q + kXcds * hl) * Tq + i0 + lane) | (key < 0 ? kCopyFlag : 0u);
          list[2 * pos + 1] = (uint32_t)key;
        }
      }
    }
    return;
  }
  for (int r = tid; r < rows; r += kOrderThreads) {
    const int key = key_of(r);
    const uint32_t pos = atomicAdd(&bins[bin_of(order_major(key, sc), r / Tq)], 1u);
    list[2 * pos] = (uint32_t)global_row(r) | (key < 0 ? kCopyFlag : 0u);
    list[2 * pos + 1] = (uint32_t)key;
  }
}

// One atomic increment per wave, by lane 0 only; returns the counter's previous value, wave-uniform.  Written as assembly
// around an exec-mask switch, not as `if (lane == 0) atomicAdd(...)`: a value that stays live across loop iterations
// inside a lane-dependent branch makes the compiler treat the whole scheduling state of the kernel as lane-dependent.
// The wait is part of the statement: the compiler takes an output for written when the statement ends and may copy or
// spill its register, which an increment still in flight would make a copy of something else.  It costs nothing, since every
// place that draws a ticket waits for all of the wave's requests right behind it.
__device__ __forceinline__ unsigned sa_lane0_atomic_inc(uint32_t* counter) {
  unsigned old, value;
  unsigned long long saved;
  asm volatile(
      "s_mov_b64 %1, exec\n\ts_mov_b64 exec, 1\n\tglobal_atomic_add %0, %3, %4, %5 sc0\n\ts_mov_b64 exec, %1\n\t"
      "s_waitcnt vmcnt(0)\n\tv_readfirstlane_b32 %2, %0"
      : "=&v"(old), "=&s"(saved), "=&s"(value)
      : "v"(0u), "v"(1u), "s"(counter)
      : "memory");
  return value;
}
// The same for a counter that goes from `last` back to 0.
__device__ __forceinline__ unsigned sa_lane0_atomic_inc_wrap(uint32_t* counter, unsigned last) {
  unsigned old, value;
  unsigned long long saved;
  asm volatile(
      "s_mov_b64 %1, exec\n\ts_mov_b64 exec, 1\n\tglobal_atomic_inc %0, %3, %4, %5 sc0\n\ts_mov_b64 exec, %1\n\t"
      "s_waitcnt vmcnt(0)\n\tv_readfirstlane_b32 %2, %0"
      : "=&v"(old), "=&s"(saved), "=&s"(value)
      : "v"(0u), "v"(last), "s"(counter)
      : "memory");
  return value;
}
// The lane number, formed where it is needed: offsets that follow from it are then not computed once, in front of the item
// loop, to occupy registers for the whole kernel (the instance for 33024 tokens of 128 channels takes 229 vector registers; with the
// lane number computed once it takes all 256 and spills 13).
__device__ __forceinline__ int sa_fresh_lane() {
  int ln;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
  return ln;
}
// A work-list entry (two words) read with one scalar load instead of a vector load and a lane broadcast.  Load and
// wait are one statement on purpose: the compiler does not know that the result arrives late and may copy the
// registers in between.
__device__ __forceinline__ unsigned long long sa_scalar_load_b64(const uint32_t* ptr) {
  unsigned long long v;
  asm volatile("s_load_dwordx2 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(v) : "s"(ptr) : "memory");
  return v;
}

// Buffer descriptor of `bytes` bytes at `base` (both wave-uniform): reads past the end give zeros.  A lane reads past it if its
// offset, lane register and instruction field, is not below `bytes` less the scalar offset; a scalar offset past the end would
// leave that difference to how it wraps.
__device__ __forceinline__ u32x4 sa_buffer(const char* base, unsigned bytes) {
  const unsigned long long a = (unsigned long long)base;
  u32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((unsigned)a);
  r[1] = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32)) & 0xffffu;   // stride 0
  r[2] = bytes;
  r[3] = 0x00020000u;                                                     // raw buffer of 32-bit words
  return r;
}
// Direct-to-LDS load through a buffer descriptor: every lane fetches 16 bytes at lane_off + tile_off + DT of the buffer, the
// wave's 1 KiB lands at lds_addr + LDS0 + DT; lanes past the end of the buffer write zeros.  The distance of the
// loads of a tile is the same in memory and in LDS, so what fits the instruction's offset field (it moves both addresses)
// goes there, and M0 is formed from one register: no address sits in a register of its own.  In assembly for the reason
// given at sa_load_to_lds_16B; the wait state behind the write of M0 is the addition that forms an offset, where there is one.
// CHECKED: the tile may reach past the end of the buffer.  It starts inside, so with all of the distance in the lane's offset the
// scalar offset stays inside too.  The lane's offsets with a distance are formed once per kernel, in two to six registers (an
// addition for each load, in the place of the wait state, took 219.0 us instead of 217.1 with 24 heads of 64, 9001 tokens, 40 % keep,
// 25 % cached).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int LDS0, int DT, bool CHECKED>
__device__ __forceinline__ void sa_tile_to_lds(const u32x4& buffer, unsigned lane_off, unsigned tile_off, unsigned lds_addr) {
  constexpr int HI = DT / 4096 * 4096, LO = DT % 4096;
  if constexpr (CHECKED || HI == 0) {
    asm volatile("s_add_u32 m0, %0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen offset:%5 lds"
                 :
                 : "s"(lds_addr), "v"(lane_off + HI), "s"(buffer), "s"(tile_off), "i"(LDS0 + HI), "i"(LO)
                 : "memory", "m0", "scc");
  } else {
    unsigned off;
    asm volatile("s_add_u32 m0, %1, %5\n\ts_add_u32 %0, %4, %7\n\tbuffer_load_dwordx4 %2, %3, %0 offen offset:%6 lds"
                 : "=&s"(off)
                 : "s"(lds_addr), "v"(lane_off), "s"(buffer), "s"(tile_off), "i"(LDS0 + HI), "i"(LO), "i"(HI)
                 : "memory", "m0", "scc");
  }
}
#pragma clang diagnostic pop

// ---------------------------------------------------------------------------------------
// LDS layouts.  A sub-tile is KEYS rows of D bf16, row major, with the 16-byte chunks of a
// row permuted by an XOR that depends on the row, so that (a) the 32 rows x 16 B that one
// S^T operand read touches and (b) the 8 rows x 64 B that one transposed V read touches fall
// into distinct banks.  A direct-to-LDS load writes 1 KiB of consecutive LDS per wave
// instruction, so the permutation is applied to the global address each lane fetches.
// ---------------------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ int k_swizzle(int row) {
  return D == 128 ? (row & 15) : ((row >> 1) & 7);
}
template <int D>
__device__ __forceinline__ int v_swizzle(int row) {
  return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1);
}

// RAGGED: the sequence length is not a multiple of the blocks (Definition 1 counts ceil(L / b) of them).
// The last query block then has fewer rows and the last key block fewer keys: missing K and V rows are zeros
// (range check of the buffer loads), scores of missing keys are set to -inf before the softmax, stores of
// missing query rows are dropped, and a sub-tile that lies entirely past the end is not visited.
// The aligned instantiation contains none of this.
// KEYS: keys per sub-tile.  MODE: how the rows get to the workgroups.
template <int D, int BQ, int BK, int KEYS, bool RAGGED, int MODE>
__global__ void __launch_bounds__(BQ * 2, attn_waves_per_simd(D, MODE)) attn_kernel(const AttnParams p) {
  constexpr bool DEALT = MODE == kDealt, SORTED = MODE == kSorted;
  constexpr int NWAVES = BQ / 32;
  constexpr int NT = NWAVES * 64;
  constexpr int SUB = BK / KEYS;           // LDS sub-tiles per symbol bit
  constexpr int CH = D / 8;                // 16-byte chunks per row
  constexpr int ROWB = D * 2;              // bytes per row
  constexpr int TILEB = KEYS * ROWB;      // bytes per K or V sub-tile
  constexpr int NINST = TILEB / 1024;      // direct-to-LDS wave instructions per sub-tile
  constexpr int NLOAD = NINST / NWAVES;    // of which this wave issues
  constexpr int ROWS_PER_INST = 1024 / ROWB;
  constexpr int KS = D / 16;               // k-steps of the S^T product
  constexpr int DB = D / 32;               // 32-row blocks of O^T
  constexpr int NQK = KEYS / 32 * KS;      // MFMAs of S^T per sub-tile
  constexpr int NPV = KEYS / 16 * DB;      // MFMAs of O^T per sub-tile
  constexpr int kPre = 4;                  // operand reads run this many MFMAs ahead
  static_assert(NINST % NWAVES == 0, "sub-tile loads must split evenly over the waves");

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  char* const ldsK = smem;                 // two K sub-tiles, then two V sub-tiles
  char* const ldsV = smem + 2 * TILEB;
  LDS_PTR(volatile int) const s_item = (LDS_PTR(volatile int))(smem + 4 * TILEB);

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned lds_wave = (unsigned)(uintptr_t)(LDS_PTR(char))smem + (unsigned)wave * 1024u;   // where its loads go
  const int l32 = lane & 31;    // query row inside the wave's 32-row slab / key row of an operand read
  const int half = lane >> 5;   // which 8 of the 16 k-slots of an MFMA this lane feeds
  const int i16 = lane & 15;
  const int g4 = lane >> 4;
  const float score_scale = p.scale_log2;

  // Per-lane offsets, the same for every item.
  // Global byte offsets inside a sub-tile (swizzle applied to the source).  Load t of a wave lies t * NWAVES KiB behind its
  // first, in memory and in LDS; the swizzles repeat every 16 rows, so up to that the lane offsets of load t and t + TP agree.
  constexpr int TP = NWAVES * ROWS_PER_INST >= 16 ? 1 : 16 / (NWAVES * ROWS_PER_INST);
  static_assert(NLOAD % TP == 0, "loads of a wave must be whole swizzle periods");
  unsigned k_goff[TP], v_goff[TP];
#pragma unroll
  for (int t = 0; t < TP; ++t) {
    const int r = (wave + t * NWAVES) * ROWS_PER_INST + lane / CH;
    const int pch = lane % CH;
    k_goff[t] = (unsigned)(r * ROWB + ((pch ^ k_swizzle<D>(r)) * 16) - t * NWAVES * 1024);
    v_goff[t] = (unsigned)(r * ROWB + ((pch ^ v_swizzle<D>(r)) * 16) - t * NWAVES * 1024);
  }
  int k_off[KS];     // S^T operand (K rows): LDS byte offset of k-step ks inside this lane's key row
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) k_off[ks] = l32 * ROWB + (((2 * ks + half) ^ k_swizzle<D>(l32)) * 16);
  int v_off[DB];     // O^T operand (V transposed): LDS byte offset of d-block db for this lane
  {
    const int r = 4 * (g4 >> 1) + (i16 >> 2);   // key row inside an 8-row group; rows +8, +16, ... share the swizzle
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      const int ch = 4 * db + 2 * (g4 & 1) + ((i16 & 3) >> 1);
      v_off[db] = r * ROWB + ((ch ^ v_swizzle<D>(r)) * 16) + 8 * (i16 & 1);
    }
  }

  // Work acquisition.
  // DEALT: the eight XCDs (workgroup n runs on XCD n mod 8) own a contiguous part each of the rows, and a workgroup
  // takes every nwg-th of its XCD's part.
  // Queues: the queue of XCD q holds its rows at list positions queue_begin(q) .. queue_begin(q + 1) - 1.  The first
  // nwg(q) of them are the first items of the workgroups n = q, q + 8, ...; the ticket of every further item is one
  // atomic on the home queue -- the one of the XCD the workgroup runs on (hardware register XCC_ID) --, issued by wave
  // 0 a few kept blocks before the current item ends (earlier would let an idle workgroup find the queue empty while
  // this one still sits on an item it has not started), where it waits for its requests anyway, so that at the end of
  // the item the ticket is there.  When the home queue is drained the workgroup looks at all queue heads at once and
  // steals from the next one that has rows left (heads only grow: one that is seen drained stays so).
  // The item number reaches the other waves through one of two LDS slots, used in turn: a wave reads slot s of item i
  // before it arrives at the barrier of item i + 1, and the slot is not written again before that barrier has been
  // passed, so one barrier per item is enough.  The barrier waits for LDS traffic only; __syncthreads() would also
  // make every wave wait for the acknowledgement of its stores of the previous item.  The work-list entry then comes
  // through the scalar cache and carries the row's kept-block count and first kept block, so the first K/V sub-tile
  // is requested before the row's symbol words have been looked at.
  const int my_q = (int)(__builtin_amdgcn_s_getreg(kHwRegXccId) & 15u) % kXcds;
  uint32_t* const q_head = p.queues;
  auto nwg = [&](int q) -> int { return ((int)gridDim.x - q + kXcds - 1) / kXcds; };
  auto queue_begin = [&](int q) -> int { return queue_first_head(q, p.BH) * p.Tq; };
  // Workgroups s and s + kCusPerXcd of an XCD share a CU.  A list starts with its longest rows, longest first, so the
  // first kCusPerXcd of them are handed out backwards: the CUs whose second workgroup comes away empty or with a
  // short row then have the longest ones, and the sums are even where a list has one or two rows per CU.
  auto first_of = [&](int q0, int slot) -> int {
    const int chunk = slot / kCusPerXcd * kCusPerXcd;
    const bool back = (slot / kCusPerXcd) % 2 == 0 && chunk + kCusPerXcd <= nwg(q0);
    return back ? 2 * chunk + kCusPerXcd - 1 - slot : slot;
  };
  int W = 0;                           // SORTED: workgroups of this XCD
  // SORTED.  After the first round the rows go to the workgroups from the end, the shortest row's first, except in a last round
  // that does not reach all of them: there to those launched first, whose waves issue first and which are done first, while the
  // others still run.  Of four two-wave workgroups on a CU each shares a SIMD with the one launched before it and one with the one
  // launched after it (read from HW_ID), so the first and the third are taken before the second; where more than these have a
  // second row the shortest ones' are better.  24 heads, keep and cached share, us, work list / from the end / this: 64 channels in
  // 64 x 128 blocks, 3584 tokens, 90 % 109 / 116 / 102; 4096, 90 % 128 / 136 / 123, 50 % 87 / 82 / 75; 4608, 90 % and 30 % 131 / 140 / 119;
  // 128 channels in 128-row blocks, 3500 tokens, 90 % 156 / 152 / 145; 4608, 30 % and 30 % 82 / 81 / 73.
  auto early_of = [&](int slot) -> int {
    if (W != 4 * kCusPerXcd) return slot;
    const int c = slot / kCusPerXcd;
    return (c == 1 ? 2 : c == 2 ? 1 : c) * kCusPerXcd + slot % kCusPerXcd;
  };
  uint32_t* const sort_keys = (uint32_t*)(smem + 4 * TILEB + 16);
  uint32_t* const sort_list = sort_keys + kSortRows;
  uint32_t* const sort_words = sort_list + kSortRows;
  uint32_t* const sort_computed = sort_words + kSortRows * kSortWords;
  int list_at = -1, list_round = 0, copy_at = 0, copy_step = 1, copy_end = 0, rest_at = 0, n_computed = 0, n_list = 0;
  if constexpr (SORTED) {
    const int q0 = (int)blockIdx.x % kXcds, slot = (int)blockIdx.x / kXcds;
    const int row0 = q0 * (p.N / kXcds) + min(q0, p.N % kXcds), rows = p.N / kXcds + (q0 < p.N % kXcds ? 1 : 0);
    const int tid = (int)threadIdx.x;
    if (tid == 0) *sort_computed = 0u;
    for (int r = tid; r < (rows + 3) / 4 * 4; r += NT) {
      uint32_t k = 0u;
      if (r < rows) {
        const unsigned flag = p.raw_flags ? p.raw_flags[row0 + r] : 0u;
        // rows start at any byte: aligned words, shifted together; only words that hold a byte of the row are read
        const uint8_t* src = p.raw_mask + (size_t)(row0 + r) * p.raw_row_bytes;      // (these calls have a mask)
        const int skew = (int)((uintptr_t)src & 3);
        const uint32_t* aligned = (const uint32_t*)(src - skew);
        const int last = (skew + p.raw_row_bytes - 1) / 4;
        uint32_t low = aligned[0];
        int count = 0;
#pragma unroll
        for (int w = 0; w < kSortWords; ++w) {
          const uint32_t high = aligned[min(w + 1, last)];
          uint32_t word = (uint32_t)(((unsigned long long)high << 32 | low) >> (8 * skew));
          word = __builtin_bswap32(__brev(word));       // most significant bit first inside each byte
          word = w < p.nw32 ? clear_padding(word, w, p.Tkv) : 0u;
          sort_words[r * kSortWords + w] = word;
          count += __popc(word);
          low = high;
        }
        // computed rows above cached ones, more kept blocks above fewer, earlier rows above later ones
        k = (flag ? 0u : (uint32_t)(count + 1) << 16) | (uint32_t)(rows - 1 - r);
      }
      sort_keys[r] = k;
    }
    __syncthreads();
    for (int r = tid; r < rows; r += NT) {
      const uint32_t k = sort_keys[r];
      int rank = 0;
      for (int i = 0; i < rows; i += 4) {
        const u32x4 o = *(const u32x4*)(sort_keys + i);
        rank += (o[0] > k) + (o[1] > k) + (o[2] > k) + (o[3] > k);
      }
      sort_list[rank] = k;
      if (k >> 16) atomicAdd(sort_computed, 1u);
    }
    __syncthreads();
    n_list = rows;
    n_computed = __builtin_amdgcn_readfirstlane((int)*sort_computed);
    W = nwg(q0);
    list_at = first_of(q0, slot);
    if (p.n_terms > 0 || p.do_copy) {
      // Cached rows: workgroups without a computed one take some each, as many as fit beside the longest computed row; the others
      // are dealt to all.  Moving a row is taken to last as long as three blocks of one; a call's time is the same for one to
      // three and grows beyond (24 heads, us, 1 / 3 / 6 / 12 blocks: 4608 tokens, 30 % keep, 56 % cached 50.8 / 50.9 / 50.7 / 54.7; 6000,
      // 20 % and 90 % 48.5 / 48.5 / 49.7 / 52.5; 64 channels, 64-row blocks, 4608, 10 % and 90 % 26.0 / 26.0 / 27.2 / 28.0).
      const int cached = rows - n_computed, idle = max(0, W - n_computed);
      const int each = max(1, (int)(__builtin_amdgcn_readfirstlane((int)sort_list[0]) >> 16) / 3);
      const int by_idle = min(cached, idle * each);
      if (list_at >= n_computed) {
        copy_at = list_at - n_computed;
        copy_step = idle;
        copy_end = by_idle;
      }
      rest_at = by_idle + (idle ? slot : W - 1 - slot);
    } else {
      n_list = n_computed;
      rest_at = rows;
    }
  }
  int next_n;                          // DEALT: next row; queues: the first item
  {
    const int q0 = (int)blockIdx.x % kXcds, slot = (int)blockIdx.x / kXcds;
    if constexpr (SORTED) {
      next_n = 0;
    } else if constexpr (DEALT) {
      next_n = slot + q0 * (p.N / kXcds) + min(q0, p.N % kXcds);
    } else {
      next_n = queue_begin(q0) + first_of(q0, slot);
      if (next_n >= queue_begin(q0 + 1)) next_n = -1;
    }
  }
  constexpr int kDrawTiles = 6;        // kept blocks an item still has to visit when the next ticket is drawn
  bool drawn = false, first_item = true;
  unsigned ticket = 0;                 // wave 0: the ticket of the home queue, where `drawn`
  auto draw_issue = [&]() {
    if constexpr (MODE == kQueues) {
      if (wave == 0) ticket = sa_lane0_atomic_inc(q_head + my_q * kHeadStride);   // a drained queue just keeps counting
      drawn = true;
    }
  };
  for (int parity = 0;; parity ^= 1) {
    int n = next_n;
    if constexpr (SORTED) {
      // computed rows in turn from both ends of the workgroups, then cached ones
      const int slot = (int)blockIdx.x / kXcds;
      if (list_at < n_computed) {
        n = list_at;
        ++list_round;
        const int left = n_computed - list_round * W;
        const bool from_end = left >= W ? list_round % 2 == 1 : W == 4 * kCusPerXcd && left > W / 2;
        list_at = list_round * W + (from_end ? W - 1 - slot : early_of(slot));
      } else if (copy_at < copy_end) {
        n = n_computed + copy_at;
        copy_at += copy_step;
      } else {
        n = n_computed + rest_at;
        rest_at += W;
        if (n >= n_list) break;
      }
      if (!first_item) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the LDS buffers are free
    } else if constexpr (DEALT) {
      const int q0 = (int)blockIdx.x % kXcds;
      if (n >= (q0 + 1) * (p.N / kXcds) + min(q0 + 1, p.N % kXcds)) break;
      if (!first_item) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the LDS buffers are free
      next_n = n + nwg(q0);
    } else if (!first_item || n < 0) {
      if (!drawn) draw_issue();
      if (wave == 0) {
        // resolve the ticket, or steal (a head counts at most the items and one overshoot per workgroup)
        int item = queue_begin(my_q) + nwg(my_q) + (int)ticket;
        if (item >= queue_begin(my_q + 1)) item = -1;
        const int ln = sa_fresh_lane();
        unsigned drained = 0;          // queues an increment of this workgroup found empty: at most eight rounds fail
        while (item < 0) {
          const int q = (my_q + ln) % kXcds;       // lanes 0..7: the eight queues, the home queue first
          const int room = queue_begin(q + 1) - queue_begin(q) - nwg(q);
          const int taken = (int)__hip_atomic_load(q_head + q * kHeadStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          const unsigned long long open = __builtin_amdgcn_ballot_w64(ln < kXcds && taken < room && !((drained >> q) & 1u));
          if (open == 0ull) break;
          const int qs = (my_q + __builtin_ctzll(open)) % kXcds;
          const int got = queue_begin(qs) + nwg(qs) + (int)sa_lane0_atomic_inc(q_head + qs * kHeadStride);
          if (got < queue_begin(qs + 1)) item = got;
          drained |= 1u << qs;
        }
        s_item[parity] = item;         // every lane writes the same value
      }
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      n = __builtin_amdgcn_readfirstlane(s_item[parity]);
      if (n < 0) break;
    }
    drawn = false;
    first_item = false;
    // Q fragment: B operand of S^T = K Q^T; lane holds query row l32, d = 16*ks + 8*half .. +7, exactly as stored:
    // the products accumulate in fp32 and the scale log2(e)/sqrt(D) is applied to the fp32 score on its way into
    // the exponential (scaling the fragment instead would save that multiply but round the queries a second time).
    bf16x8 qf[KS];
    auto load_q = [&](size_t off, int block) {
      const int ln = sa_fresh_lane();
      int qr = wave * 32 + (ln & 31);
      if constexpr (RAGGED) qr = min(qr, p.L - 1 - block * BQ);
      const char* qrow = p.Q + off + (size_t)qr * ROWB + (ln >> 5) * 16;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 q = *(const bf16x8*)(qrow + ks * 32);
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[ks][e] = q[e];
      }
    };
    // row, and its key: kept blocks | first kept block << 16
    uint32_t entry, key, raw_words = 0;
    if constexpr (SORTED) {
      const int q0 = (int)blockIdx.x % kXcds;
      const uint32_t k = (uint32_t)__builtin_amdgcn_readfirstlane((int)sort_list[n]);
      const int rows = p.N / kXcds + (q0 < p.N % kXcds ? 1 : 0), r = rows - 1 - (int)(k & 0xffffu);
      entry = (uint32_t)(q0 * (p.N / kXcds) + min(q0, p.N % kXcds) + r) | (k >> 16 ? 0u : kCopyFlag);
      raw_words = lane < kSortWords ? sort_words[r * kSortWords + lane] : 0u;
      const unsigned long long some = __builtin_amdgcn_ballot_w64(raw_words != 0u);
      const int w = some ? __builtin_ctzll(some) : 0;
      const uint32_t bits = (uint32_t)__builtin_amdgcn_readlane((int)raw_words, w);
      key = some ? 1u | (uint32_t)(32 * w + __builtin_ctz(bits)) << 16 : 0u;      // (the count is for queues: any, or none)
    } else if constexpr (DEALT) {
      // Symbols as the caller gave them, at most 64 words a row: lane w decodes word w.  A short call is a chain of round
      // trips to memory, so flag, symbols and queries are requested together (40 heads of 64, 1024 tokens: 12.5 -> 12.1 us).
      entry = (uint32_t)n;
      const unsigned flag = p.raw_flags ? p.raw_flags[n] : 0u;
      const bool has_word = lane < p.nw32;
      uint32_t byte[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) byte[b] = 0xffu;
      if (p.raw_mask) {
        const uint8_t* src = p.raw_mask + (size_t)n * p.raw_row_bytes;
#pragma unroll
        for (int b = 0; b < 4; ++b) byte[b] = src[min(4 * lane + b, p.raw_row_bytes - 1)];
      }
      {
        const int head = n / p.Tq, block = n - head * p.Tq;
        load_q(((size_t)head * p.L + (size_t)block * BQ) * ROWB, block);
      }
      raw_words = byte[0] | byte[1] << 8 | byte[2] << 16 | byte[3] << 24;
      // most significant bit first inside each byte; bytes past the row's last are padding
      raw_words = has_word ? clear_padding(__builtin_bswap32(__brev(raw_words)), lane, p.Tkv) : 0u;
      if (__builtin_amdgcn_readfirstlane((int)flag) != 0) entry |= kCopyFlag;
      const unsigned long long some = __builtin_amdgcn_ballot_w64(raw_words != 0u);
      const int w = some ? __builtin_ctzll(some) : 0;
      const uint32_t bits = (uint32_t)__builtin_amdgcn_readlane((int)raw_words, w);
      key = some ? 1u | (uint32_t)(32 * w + __builtin_ctz(bits)) << 16 : 0u;      // (the count is for queues: any, or none)
    } else {
      const unsigned long long entry64 = sa_scalar_load_b64(p.order + 2 * (size_t)n);
      entry = (uint32_t)entry64;
      key = (uint32_t)(entry64 >> 32);
    }
    const int row = (int)(entry & ~kCopyFlag);
    const int bh = row / p.Tq;
    const int iq = row - bh * p.Tq;
    const size_t head_off = (size_t)bh * p.L * ROWB;
    const size_t blk_off = head_off + (size_t)iq * BQ * ROWB;

    if (entry & kCopyFlag) {
      // cache-then-reuse: O_i <- cached O_i, bit exact
      int NV = BQ * ROWB / 16;
      if constexpr (RAGGED) NV = min(BQ, p.L - iq * BQ) * (ROWB / 16);
      const int first_vec = wave * 64 + sa_fresh_lane();
      if (p.n_terms > 0) {
        // forecast: fp32 sum of the scaled terms in order, rounded once to bf16
        const bf16x8* t0 = (const bf16x8*)(p.O_cache + blk_off);
        bf16x8* dst = (bf16x8*)(p.O + blk_off);
        for (int t = first_vec; t < NV; t += NT) {
          const bf16x8 a = t0[t];
          float acc[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] = p.coef[0] * (float)a[e];
          for (int d = 1; d < p.n_terms; ++d) {
            const bf16x8 b = ((const bf16x8*)(p.term[d - 1] + blk_off))[t];
            const float c = p.coef[d];
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] = fmaf(c, (float)b[e], acc[e]);
          }
          bf16x8 r;
#pragma unroll
          for (int e = 0; e < 8; ++e) r[e] = (__bf16)acc[e];
          dst[t] = r;
        }
      } else if (p.do_copy) {
        const u32x4* src = (const u32x4*)(p.O_cache + blk_off);
        u32x4* dst = (u32x4*)(p.O + blk_off);
#pragma unroll 4
        for (int t = first_vec; t < NV; t += NT) dst[t] = src[t];
      }
      continue;
    }

    // ---- compute-on-demand ----
    const u32x4 Kh = sa_buffer(p.K + head_off, (unsigned)(p.L * ROWB));      // (at most 2^21 rows of 256 bytes)
    const u32x4 Vh = sa_buffer(p.V + head_off, (unsigned)(p.L * ROWB));
    const uint32_t* wp = MODE != kQueues ? nullptr : p.words + (size_t)row * p.nw32;

    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[db][e] = 0.f;
    // Reference of the scores (raw q.k units, before the scale) of this lane's query row, kept NEGATED in all 16
    // registers of an accumulator: it is the C operand of the first MFMA of every S^T block, so
    // the MFMA delivers score - reference and the softmax needs no subtraction per score either.
    // The reference is not the running maximum: it is raised (to the row maximum seen so far) only
    // when the weights of a sub-tile show that a score left the allowed range above it; the final
    // division by the row sum cancels it exactly.
    f32x16 neg_ref;
#pragma unroll
    for (int e = 0; e < 16; ++e) neg_ref[e] = 0.f;
    bool first = true;
    bool late = false;   // 32-key sub-tiles: the even one raised the reference by late_by, the odd one has not followed yet
    float late_by = 0.f;
    float l_run = 0.f;   // per-lane partial row sum (this lane's half of the keys)

    // Scalar walk over the set bits of the decoded symbol row.  The row's words sit one per lane in a vector
    // register (one coalesced load per item, 64 words at a time), so moving on to the next word is a lane read,
    // not a memory access.
    int tiles_left = (int)(key & 0xffffu);          // kept blocks not yet visited, the current one included
    int w_idx = (int)(key >> 21);                    // word of the first kept block
    auto load_words = [&](int w0) -> uint32_t {
      if constexpr (MODE != kQueues) return raw_words;       // one word per lane, w0 == 0
      return w0 + lane < p.nw32 ? wp[w0 + lane] : 0u;
    };
    uint32_t w_lanes = load_words(w_idx & ~63);
    uint32_t w_bits = 0;
    auto next_block = [&]() -> int {
      while (w_bits == 0u) {
        ++w_idx;
        if (w_idx >= p.nw32) return -1;
        if ((w_idx & 63) == 0) w_lanes = load_words(w_idx);
        w_bits = (uint32_t)__builtin_amdgcn_readlane((int)w_lanes, w_idx & 63);
      }
      const int b = __builtin_ctz(w_bits);
      w_bits &= w_bits - 1u;
      return 32 * w_idx + b;
    };

    // load t of this wave's NLOAD for the sub-tile at byte tile_off of the head
    auto issue_load = [&](unsigned tile_off, auto buf_c, auto t_c) {
      constexpr int buf = decltype(buf_c)::value, t = decltype(t_c)::value;
      sa_tile_to_lds<buf * TILEB, t * NWAVES * 1024, RAGGED>(Kh, k_goff[t % TP], tile_off, lds_wave);
      sa_tile_to_lds<(2 + buf) * TILEB, t * NWAVES * 1024, RAGGED>(Vh, v_goff[t % TP], tile_off, lds_wave);
    };
    auto tile_offset = [&](int j, int sub) -> unsigned { return (unsigned)(j * BK + sub * KEYS) * ROWB; };

    // valid: keys of this sub-tile that exist (RAGGED only); (nj, nsub): the sub-tile to fetch into the other
    // buffer meanwhile, nj < 0 if there is none
    auto compute = [&](auto buf_c, auto other_c, int valid, int nj, int nsub) {
      // the buffer index is a compile-time constant, so every LDS address below is a per-lane
      // register that never changes plus an immediate offset
      constexpr int buf = decltype(buf_c)::value;
      const char* kb = ldsK + buf * TILEB;
      const char* vb = ldsV + buf * TILEB;
      auto k_read = [&](int t) -> bf16x8 {   // operand t = (kb2, ks)
        return *(const bf16x8*)(kb + (t / KS) * 32 * ROWB + k_off[t % KS]);
      };
      auto v_read = [&](int t) -> bf16x8 {   // operand t = ((kb2, ksp), db): keys 16*(t/DB) .. +15, d-block t%DB
        const char* base = vb + (t / DB) * 16 * ROWB + v_off[t % DB];
        const s16x4 t1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))(base));
        const s16x4 t2 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))(base + 8 * ROWB));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(t1, t2, 0, 1, 2, 3, 4, 5, 6, 7));
      };

      // A sub-tile of 64 keys is two blocks of 32 (one 32x32 S^T accumulator each).  Within this wave the
      // instruction stream is ordered so that the vector work of the softmax sits BETWEEN matrix instructions
      // that do not depend on it -- a wave's VALU instructions issue while its own earlier MFMA is still in the
      // matrix pipe, but only if they come right behind it in program order:
      //   S0:  scores of block 0                      (KS MFMAs)
      //   S1:  scores of block 1      || weights of block 0   (KS MFMAs, 32 vector instructions spread over them)
      //   PV0: O^T += V^T P^T, block 0 || weights of block 1
      //   PV1: O^T += V^T P^T, block 1
      // Weights are rounded to bf16 for the O^T product and the row sum adds up the same rounded values.
      // k-slot s of lane-half h of the O^T MFMA maps to key 32*kb2 + 16*ksp + 8*(s/4) + 4*h + s%4, which is
      // exactly the key order of the S^T accumulator registers 8*ksp .. 8*ksp+7.
      // The exponent's reference is checked after the fact, block by block: the weights are formed against
      // the current reference straight away, and only if their sum shows that one of them left the allowed
      // range is the block's row maximum taken, the reference moved and the block's weights formed again.
      constexpr int CPS = 8 / KS;     // weight chunks (two scores each) per MFMA slot of a group
      f32x16 s[2];
      bf16x8 pb[4];
      bf16x2 ones;
      ones[0] = (__bf16)1.0f;
      ones[1] = (__bf16)1.0f;
      auto chunk = [&](int kb2, int c, float& dl) {
        const int g = 2 * kb2 + c / 4, e = 2 * (c % 4);
        bf16x2 pr;
        pr[0] = (__bf16)__builtin_amdgcn_exp2f(s[kb2][8 * (g & 1) + e] * score_scale);
        pr[1] = (__bf16)__builtin_amdgcn_exp2f(s[kb2][8 * (g & 1) + e + 1] * score_scale);
        pb[g][e] = pr[0];
        pb[g][e + 1] = pr[1];
        dl = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, dl, false);
      };
      auto mask_block = [&](int kb2) {
        // accumulator register e of block kb2 is key 32*kb2 + 8*(e/4) + 4*half + e%4 of the sub-tile
        const int lim = valid - 4 * half;
#pragma unroll
        for (int e = 0; e < 16; ++e) s[kb2][e] = (32 * kb2 + 8 * (e / 4) + e % 4 >= lim) ? -INFINITY : s[kb2][e];
      };
      // Moves the reference to the row maximum of block kb2 (upwards only, except on the very first block of an
      // item, which sets it) in what has been computed against it and returns by how much; lower_reference() does the
      // same to the negated reference itself.  `other_too`: block 1's scores were formed against the old reference as well.
      auto lower_reference = [&](float d) {
        const float nr = neg_ref[0] - d;
#pragma unroll
        for (int e = 0; e < 16; ++e) neg_ref[e] = nr;
      };
      auto move_reference = [&](int kb2, bool other_too) -> float {
        float mx = s[kb2][0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[kb2][e]);
        {
          // this lane sees 16 of the 32 scores of its query row in this block; the other half sits in lane ^ 32
          const unsigned bits = __builtin_bit_cast(unsigned, mx);
          const auto sw = __builtin_amdgcn_permlane32_swap(bits, bits, false, false);
          mx = fmaxf(__builtin_bit_cast(float, (unsigned)sw[0]), __builtin_bit_cast(float, (unsigned)sw[1]));
        }
        const float d = first ? mx : fmaxf(mx, 0.f);
#pragma unroll
        for (int e = 0; e < 16; ++e) s[kb2][e] -= d;
        if (other_too) {
#pragma unroll
          for (int e = 0; e < 16; ++e) s[1][e] -= d;
        }
        if (!first) {
          const float alpha = __builtin_amdgcn_exp2f(-d * score_scale);
          l_run *= alpha;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[db][e] *= alpha;
        }
        first = false;
        return d;
      };

      bf16x8 ka[NQK];
#pragma unroll
      for (int t = 0; t < kPre; ++t) ka[t] = k_read(t);
      __builtin_amdgcn_s_setprio(kMfmaPrio);
      // ---- S0; the next sub-tile's loads go out here, a few behind each matrix instruction, instead of in one burst in
      // front of the first one.  One branch around all of it: with one per load, 64-bit addresses and an M0 value for each, the
      // scalar instructions between the matrix instructions took longer than these (24 heads, 9001 tokens at 40 % keep
      // and 25 % cached, before / after: 64 channels 225 / 211 us, 128 channels 331 / 318).
      auto s0 = [&](auto loads) {
        const unsigned next_off = tile_offset(nj, nsub);
        static_for<KS>([&](auto t_c) {
          constexpr int t = decltype(t_c)::value;
          if constexpr (t + kPre < NQK) ka[t + kPre] = k_read(t + kPre);
          s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[t], qf[t], t == 0 ? neg_ref : s[0], 0, 0, 0);
          if constexpr (decltype(loads)::value) {
            constexpr int lo = t * NLOAD / KS, hi = (t + 1) * NLOAD / KS;
            static_for<hi - lo>([&](auto i) { issue_load(next_off, other_c, std::integral_constant<int, lo + decltype(i)::value>{}); });
          }
        });
      };
      if (nj >= 0)
        s0(std::true_type{});
      else
        s0(std::false_type{});
      if constexpr (RAGGED) {
        if (valid < KEYS) mask_block(0);
      }
      if (first) lower_reference(move_reference(0, false));     // the first block of an item sets the reference; block 1 is not formed yet
      if constexpr (KEYS == 32) {
        // One block: its weights have no matrix instructions of this wave to hide under; four workgroups on the CU do.
        // Two sub-tiles (the even one in buffer 0) are rounded like the two blocks of a 64-key sub-tile, where block 1's
        // scores are formed before block 0's weights can raise the reference: a move of the even one takes effect on
        // the scores of the odd one, not on the C operand that forms them.
        if constexpr (buf == 1) {
          if (late) {
#pragma unroll
            for (int e = 0; e < 16; ++e) s[0][e] -= late_by;
            lower_reference(late_by);
            late = false;
          }
        }
        bf16x8 vv[NPV];
#pragma unroll
        for (int t = 0; t < kPre; ++t) vv[t] = v_read(t);
        float dl = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c) chunk(0, c, dl);
        if (__builtin_amdgcn_ballot_w64(!(dl <= kSumLimit)) != 0) {
          late_by = move_reference(0, false);
          if constexpr (buf == 0)
            late = true;
          else
            lower_reference(late_by);
          dl = 0.f;
#pragma unroll
          for (int c = 0; c < 8; ++c) chunk(0, c, dl);
        }
        l_run += dl;
#pragma unroll
        for (int t = 0; t < NPV; ++t) {
          if (t + kPre < NPV) vv[t + kPre] = v_read(t + kPre);
          o[t % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vv[t], pb[t / DB], o[t % DB], 0, 0, 0);
        }
      } else {
        // first operands of the O^T product: on their way while the scores of block 1 are formed
        bf16x8 va[NPV];
#pragma unroll
        for (int t = 0; t < kPre; ++t) va[t] = v_read(t);
        // ---- S1 || weights of block 0
        float dl0 = 0.f;
#pragma unroll
        for (int t = 0; t < KS; ++t) {
          if (KS + t + kPre < NQK) ka[KS + t + kPre] = k_read(KS + t + kPre);
          s[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[KS + t], qf[t], t == 0 ? neg_ref : s[1], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int cc = 0; cc < CPS; ++cc) chunk(0, t * CPS + cc, dl0);
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (RAGGED) {
          // (the sum passes through an empty asm statement in front of the branch: otherwise the compiler moves the weights
          // behind it, where no matrix instruction of this wave hides them)
          asm volatile("" : "+v"(dl0));
          if (valid < KEYS) mask_block(1);
        }
        // !(sum <= limit) also catches an overflowed (infinite or NaN) sum
        if (__builtin_amdgcn_ballot_w64(!(dl0 <= kSumLimit)) != 0) {
          lower_reference(move_reference(0, true));
          dl0 = 0.f;
#pragma unroll
          for (int c = 0; c < 8; ++c) chunk(0, c, dl0);
        }
        l_run += dl0;
        // ---- PV0 || weights of block 1
        float dl1 = 0.f;
#pragma unroll
        for (int t = 0; t < NPV / 2; ++t) {
          if (t + kPre < NPV) va[t + kPre] = v_read(t + kPre);
          o[t % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[t], pb[t / DB], o[t % DB], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int cc = 0; cc < CPS; ++cc) chunk(1, t * CPS + cc, dl1);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (__builtin_amdgcn_ballot_w64(!(dl1 <= kSumLimit)) != 0) {
          lower_reference(move_reference(1, false));
          dl1 = 0.f;
#pragma unroll
          for (int c = 0; c < 8; ++c) chunk(1, c, dl1);
        }
        l_run += dl1;
        // ---- PV1
#pragma unroll
        for (int t = NPV / 2; t < NPV; ++t) {
          if (t + kPre < NPV) va[t + kPre] = v_read(t + kPre);
          o[t % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[t], pb[t / DB], o[t % DB], 0, 0, 0);
        }
      }
      __builtin_amdgcn_s_setprio(0);
    };

    // Two sub-tiles per trip, one per LDS buffer: while sub-tile u is computed from one buffer
    // the loads of sub-tile u+1 are in flight into the other.
    using Buf0 = std::integral_constant<int, 0>;
    using Buf1 = std::integral_constant<int, 1>;
    int j = tiles_left > 0 ? (int)(key >> 16) : -1;
    int sub = 0;
    if (j >= 0) static_for<NLOAD>([&](auto t) { issue_load(tile_offset(j, 0), Buf0{}, t); });
    if constexpr (!DEALT) load_q(blk_off, iq);    // behind the first sub-tile's requests: the two latencies overlap
    // the walk continues behind the first kept block
    if (j >= 0) w_bits = (uint32_t)__builtin_amdgcn_readlane((int)w_lanes, w_idx & 63) & ~((2u << (j & 31)) - 1u);
    if (tiles_left <= kDrawTiles) draw_issue();
    auto step = [&](auto cur, auto other) {
      int nj = j, nsub = sub + 1;
      if constexpr (RAGGED) {
        if (nsub < SUB && j * BK + nsub * KEYS >= p.L) nsub = SUB;   // the rest of the last block does not exist
      }
      if (nsub == SUB) {
        nsub = 0;
        nj = next_block();
        if (--tiles_left == kDrawTiles) draw_issue();
      }
      sa_wait_vmem();
      __syncthreads();   // this sub-tile has landed for every wave; the other buffer is free
      compute(cur, other, RAGGED ? p.L - (j * BK + sub * KEYS) : KEYS, nj, nsub);
      j = nj;
      sub = nsub;
    };
    int last = 0;     // buffer of the last sub-tile
    while (j >= 0) {
      step(Buf0{}, Buf1{});
      last = 0;
      if (j < 0) break;
      step(Buf1{}, Buf0{});
      last = 1;
    }

    // O_i = diag(l)^-1 O_acc; both lane halves hold partial sums of the same row.  A lane owns one query row, so
    // stored straight from the accumulators every store instruction would touch 32 rows with 16 bytes each; the
    // block goes through LDS instead and leaves as whole rows, 16 bytes per lane.  The staging area is the buffer
    // that the last sub-tile did NOT use: nothing was fetched into it meanwhile and every wave has finished
    // reading it (it passed the barrier of the last sub-tile after that); each wave stages its own 32 rows, so
    // no barrier is needed here, and the barrier at the top of the next item comes before anything is fetched
    // into that buffer again.
    {
      const unsigned bits = __builtin_bit_cast(unsigned, l_run);
      const auto sw = __builtin_amdgcn_permlane32_swap(bits, bits, false, false);
      const float l_tot = __builtin_bit_cast(float, (unsigned)sw[0]) + __builtin_bit_cast(float, (unsigned)sw[1]);
      const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
      // (a wave's rows take 32 keys' room: K and V hold KEYS / 32 waves' each; the waves 4 to 7 of 256-row blocks have a
      // piece of LDS of their own)
      constexpr int PER = KEYS / 32;
      char* const stage = wave < 4 ? (wave < PER ? ldsK : ldsV) + (last ^ 1) * TILEB + wave % PER * 32 * ROWB
                                   : smem + 4 * TILEB + 16 + (wave - 4) * 32 * ROWB;
      const int ln = sa_fresh_lane();
      const int srow = ln & 31;
      char* const wr = stage + srow * ROWB + (ln >> 5) * 8;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          // accumulator registers 4*q4 .. 4*q4+3 hold d = 32*db + 8*q4 + 4*half + 0..3
          bf16x2 lo, hi;
          lo[0] = (__bf16)(o[db][4 * q4 + 0] * inv);
          lo[1] = (__bf16)(o[db][4 * q4 + 1] * inv);
          hi[0] = (__bf16)(o[db][4 * q4 + 2] * inv);
          hi[1] = (__bf16)(o[db][4 * q4 + 3] * inv);
          u32x2 pk;
          pk[0] = __builtin_bit_cast(unsigned, lo);
          pk[1] = __builtin_bit_cast(unsigned, hi);
          // 16-byte chunks of a row permuted by the row, so that the 32 rows of one write fall into distinct banks
          *(u32x2*)(wr + (((4 * db + q4) ^ (srow & (CH - 1))) * 16)) = pk;
        }
      constexpr int RPI = 1024 / ROWB;       // rows per store instruction
      char* const obase = p.O + blk_off + (size_t)(wave * 32) * ROWB;
      const int rows_here = RAGGED ? p.L - (iq * BQ + wave * 32) : 32;   // rows of this wave's slab that exist
#pragma unroll
      for (int t = 0; t < 32 / RPI; ++t) {
        const int r = t * RPI + ln / CH, ch = ln % CH;
        const u32x4 v = *(const u32x4*)(stage + r * ROWB + ((ch ^ (r & (CH - 1))) * 16));
        if (!RAGGED || r < rows_here) *(u32x4*)(obase + r * ROWB + ch * 16) = v;
      }
    }
  }
  if constexpr (MODE == kQueues) {
    // Stored plans: the last workgroup to get here leaves the queue heads as the next run wants them.  Every
    // workgroup has waited for its last ticket, so no increment is still on its way.  The counter of workgroups that
    // are done wraps by itself: it stays in step with the launches even where a program lets two runs of a plan overlap
    // (their outputs are wrong then), and behind the last workgroup of both it and the heads are zero again.
    if (p.self_reset && wave == 0) {
      const unsigned last = gridDim.x - 1;
      if (sa_lane0_atomic_inc_wrap(q_head + kDoneOffset, last) == last && lane < kXcds)
        __hip_atomic_store(q_head + lane * kHeadStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// ---------------------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------------------
thread_local char g_err[512] = "";

}  // namespace

int sa_fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof g_err, fmt, ap);
  va_end(ap);
  return code;
}

namespace {

#define fail sa_fail

#define HIP_TRY(expr)                                                                          \
  do {                                                                                         \
    hipError_t e_ = (expr);                                                                    \
    if (e_ != hipSuccess) return fail(SPARSE_ATTN_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

struct Shape {
  int B, H, L, D, bq, bk, Tq, Tkv, N, row_bytes, nw32;
};

int check_shape(int B, int H, int L, int D, int bq, int bk, bool need_d, Shape* s) {
  if (B <= 0 || H <= 0 || L <= 0 || bq <= 0 || bk <= 0 || (need_d && D <= 0))
    return fail(SPARSE_ATTN_ERR_INVALID, "sizes must be positive (B=%d H=%d L=%d D=%d block_q=%d block_k=%d)", B, H,
                L, D, bq, bk);
  if ((bq != 64 && bq != 128) || (bk != 64 && bk != 128))
    return fail(SPARSE_ATTN_ERR_UNSUPPORTED, "block_q and block_k must be 64 or 128 (got %d, %d)", bq, bk);
  if (need_d && D != 64 && D != 128) return fail(SPARSE_ATTN_ERR_UNSUPPORTED, "D must be 64 or 128 (got %d)", D);
  const int tq = (L + bq - 1) / bq;      // a short last block counts as a block
  const long long n = (long long)B * H * tq;
  if (tq > kMaxTq) return fail(SPARSE_ATTN_ERR_UNSUPPORTED, "Tq=%d exceeds %d", tq, kMaxTq);
  if (n > 0x3fffffffLL) return fail(SPARSE_ATTN_ERR_UNSUPPORTED, "too many query blocks (%lld)", n);
  s->B = B; s->H = H; s->L = L; s->D = D; s->bq = bq; s->bk = bk;
  s->Tq = tq;
  s->Tkv = (L + bk - 1) / bk;
  s->N = (int)n;
  s->row_bytes = (s->Tkv + 7) / 8;
  s->nw32 = (s->Tkv + 31) / 32;
  return 0;
}

// scratch layout: [queue heads (kQueueBytes)] [order N x 2 u32] [keys N i32] [words N*nw32 u32]
size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
constexpr size_t kQueueBytes = (size_t)kQueueWords * 4;
size_t workspace_bytes(const Shape& s) {
  return kQueueBytes + align256((size_t)s.N * 8) + align256((size_t)s.N * 4) + align256((size_t)s.N * s.nw32 * 4);
}

struct Scratch {
  void* ptr = nullptr;
  size_t bytes = 0;
};
std::mutex g_mu;
std::map<std::pair<int, void*>, Scratch> g_scratch;

}  // namespace

// Scratch of the entry point that allocates nothing: every GPU the library runs on holds its own copy of this
// array for the life of the process.  In host code the name is only a handle for hipGetSymbolAddress; kernels
// and copies use the per-device address that call returns.
constexpr size_t kStaticScratchBytes = SPARSE_ATTN_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
void* g_static_scratch[kMaxDevices] = {};

// Address of `scratch` on the current device, looked up once per device.
int static_scratch_ptr(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return sa_fail(SPARSE_ATTN_ERR_HIP, "hipGetDevice failed: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return sa_fail(SPARSE_ATTN_ERR_UNSUPPORTED, "device index %d is out of range", dev);
  std::lock_guard<std::mutex> lock(g_mu);
  if (!g_static_scratch[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return sa_fail(SPARSE_ATTN_ERR_HIP, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
    g_static_scratch[dev] = ptr;
  }
  *out = g_static_scratch[dev];
  return 0;
}

}  // namespace

int sa_get_scratch(size_t need, hipStream_t stream, void** out) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lock(g_mu);
  Scratch& sc = g_scratch[std::make_pair(dev, (void*)stream)];
  if (sc.bytes < need) {
    if (sc.ptr) {
      HIP_TRY(hipStreamSynchronize(stream));
      HIP_TRY(hipFree(sc.ptr));
      sc.ptr = nullptr;
      sc.bytes = 0;
    }
    const size_t want = need + need / 2;
    HIP_TRY(hipMalloc(&sc.ptr, want));
    sc.bytes = want;
  }
  *out = sc.ptr;
  return 0;
}

namespace {

// Optional per-call event recording (sparse_attn_profile_begin/end): three events per call,
// recorded on the call's stream without any synchronisation.
struct Profile {
  bool on = false;
  int capacity = 0;
  int calls = 0;
  hipEvent_t* ev = nullptr;   // 3 per call: start, after the pre-pass, end
};
Profile g_prof;

bool overlaps(const void* a, const void* b, size_t bytes) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + bytes && y < x + bytes;
}

// four K / V sub-tiles, two item slots, output rows of the waves beyond four
constexpr size_t attn_lds(int D, int bq, int keys, int mode) {
  return 4 * (size_t)keys * D * 2 + 16 + (bq > 128 ? (size_t)(bq - 128) * D * 2 : 0) + (mode == kSorted ? kSortLds : 0);
}

template <int D, int BQ, int BK, int KEYS, bool RAGGED, int MODE>
int launch_attn_variant(const AttnParams& p, int grid, hipStream_t stream) {
  constexpr size_t lds = attn_lds(D, BQ, KEYS, MODE);
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [] {
    attr_err = hipFuncSetAttribute((const void*)attn_kernel<D, BQ, BK, KEYS, RAGGED, MODE>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  });
  if (attr_err != hipSuccess)
    return fail(SPARSE_ATTN_ERR_HIP, "hipFuncSetAttribute failed: %s", hipGetErrorString(attr_err));
  hipLaunchKernelGGL((attn_kernel<D, BQ, BK, KEYS, RAGGED, MODE>), dim3(grid), dim3(BQ * 2), lds, stream, p);
  HIP_TRY(hipGetLastError());
  return 0;
}

template <int D, int BQ, int BK, int KEYS = 64>
int launch_attn(const AttnParams& p, int grid, hipStream_t stream) {
  const bool ragged = p.L % BQ || p.L % BK;
  auto go = [&](auto mode) -> int {
    constexpr int MODE = decltype(mode)::value;
    return ragged ? launch_attn_variant<D, BQ, BK, KEYS, true, MODE>(p, grid, stream)
                  : launch_attn_variant<D, BQ, BK, KEYS, false, MODE>(p, grid, stream);
  };
  if (p.mode == kQueues) return go(std::integral_constant<int, kQueues>{});
  if constexpr (BQ <= 128) {
    if (p.mode == kSorted) return go(std::integral_constant<int, kSorted>{});
  }
  return go(std::integral_constant<int, kDealt>{});
}

struct PlanBuffers {
  uint32_t* queues;   // queue heads (kQueueWords)
  uint32_t* order;    // [N][2]
  int32_t* keys;      // [N]
  uint32_t* words;    // [N][nw32]
};

PlanBuffers carve(char* base, const Shape& s) {
  PlanBuffers b;
  b.queues = (uint32_t*)base;
  b.order = (uint32_t*)(base + kQueueBytes);
  b.keys = (int32_t*)(base + kQueueBytes + align256((size_t)s.N * 8));
  b.words = (uint32_t*)(base + kQueueBytes + align256((size_t)s.N * 8) + align256((size_t)s.N * 4));
  return b;
}

}  // namespace

// A stored pre-pass: decoded symbol words and the ordered work list of one set of symbols.  A run needs no other launch
// than the attention kernel: its last workgroup leaves the queue heads at zero for the next one.
struct sparse_attn_plan {
  Shape s;
  int gran;
  bool some_cached;        // the plan has cache flags
  int dev;
  void* mem;               // workspace as carved above; the queue heads are zero between runs
  PlanBuffers bufs;
};

namespace {

// Enqueues the symbol pre-pass: decode + count per row, the ordered work list, queue heads at zero.
int launch_plan(const uint8_t* cache_flags, const uint8_t* kv_mask, const Shape& s, int gran, const PlanBuffers& pb,
                hipStream_t stream) {
  const int BH = s.B * s.H;
  const int heads_per_xcd = (BH + kXcds - 1) / kXcds;
  int shift = 0;
  while (((heads_per_xcd - 1) >> shift) + 1 > kMaxHeadGroups) ++shift;
  const int groups = ((heads_per_xcd - 1) >> shift) + 1;
  const int sym_Tq = (s.Tq + gran - 1) / gran;
  const int sym_row_bytes = ((s.Tkv + gran - 1) / gran + 7) / 8;
  // A queue's workgroup decodes its rows with one thread per row, which is quickest while a queue has few words: many words
  // through one CU, each lane at a row of its own, are slow, and then a kernel over all rows decodes first.  Creating a
  // plan, us, without / with it: 2115 words in a queue 10 / 14, 6966: 15 / 15, 8772: 19 / 16, 26316: 35 / 18, 131072 (one head
  // of 131072 tokens in blocks of 64): 194 / 31; bit by bit at granularity 2: 639 words 16 / 17, 6966: 59 / 18.
  const bool decoded = (long long)heads_per_xcd * s.Tq * s.nw32 > (gran == 1 ? 8192 : 1024);
  if (decoded) {
    hipLaunchKernelGGL(decode_rows, dim3((s.N + 15) / 16), dim3(256), 0, stream, cache_flags, kv_mask, s.N, s.Tq, s.Tkv, gran,
                       sym_Tq, sym_row_bytes, s.nw32, pb.words, pb.keys);
    HIP_TRY(hipGetLastError());
  }
  hipLaunchKernelGGL(plan_queues, dim3(kXcds), dim3(kOrderThreads), 0, stream, cache_flags, kv_mask, BH, s.Tq, s.Tkv, gran,
                     sym_Tq, sym_row_bytes, s.nw32, shift, groups, decoded, pb.words, pb.keys, pb.order, pb.queues);
  HIP_TRY(hipGetLastError());
  return 0;
}

struct Forecast {
  const void* const* terms;   // host array of n device pointers
  const float* coef;          // host array of n weights
  int n;
};

int run(const void* Q, const void* K, const void* V, const uint8_t* cache_flags, const uint8_t* kv_mask,
        const void* O_cache, void* O, int B, int H, int L, int D, int bq, int bk, hipStream_t stream, float* plan_ms,
        float* attn_ms, bool timed, const Forecast* fc = nullptr, const sparse_attn_plan* plan = nullptr,
        bool static_scratch = false, void* user_ws = nullptr, size_t user_ws_bytes = 0, bool use_user_ws = false) {
  Shape s;
  if (int rc = check_shape(B, H, L, D, bq, bk, true, &s)) return rc;
  if (!Q || !K || !V || !O) return fail(SPARSE_ATTN_ERR_INVALID, "Q, K, V and O must not be NULL");
  const size_t tensor_bytes = (size_t)B * H * L * D * 2;
  if (overlaps(O, Q, tensor_bytes) || overlaps(O, K, tensor_bytes) || overlaps(O, V, tensor_bytes))
    return fail(SPARSE_ATTN_ERR_INVALID, "O must not overlap Q, K or V");
  if (O_cache && O_cache != O && overlaps(O, O_cache, tensor_bytes))
    return fail(SPARSE_ATTN_ERR_INVALID, "O_cache must be O itself or must not overlap O");
  if (((uintptr_t)Q | (uintptr_t)K | (uintptr_t)V | (uintptr_t)O | (uintptr_t)O_cache) & 15)
    return fail(SPARSE_ATTN_ERR_INVALID, "tensor base pointers must be 16-byte aligned");
  if (fc) {
    if (fc->n < 1 || fc->n > kMaxTerms)
      return fail(SPARSE_ATTN_ERR_UNSUPPORTED, "n_terms=%d must be between 1 and %d", fc->n, kMaxTerms);
    if (!fc->terms || !fc->coef) return fail(SPARSE_ATTN_ERR_INVALID, "O_terms and coef must not be NULL");
    for (int d = 0; d < fc->n; ++d) {
      if (!fc->terms[d]) return fail(SPARSE_ATTN_ERR_INVALID, "O_terms[%d] must not be NULL", d);
      if ((uintptr_t)fc->terms[d] & 15) return fail(SPARSE_ATTN_ERR_INVALID, "O_terms[%d] must be 16-byte aligned", d);
      if (overlaps(O, fc->terms[d], tensor_bytes)) return fail(SPARSE_ATTN_ERR_INVALID, "O_terms[%d] must not overlap O", d);
      if (!(fc->coef[d] == fc->coef[d]) || fc->coef[d] - fc->coef[d] != 0.f)
        return fail(SPARSE_ATTN_ERR_INVALID, "coef[%d] must be finite", d);
    }
  }

  if (use_user_ws) {
    const size_t need = workspace_bytes(s);
    if (!user_ws) return fail(SPARSE_ATTN_ERR_INVALID, "workspace must not be NULL");
    if ((uintptr_t)user_ws & 255) return fail(SPARSE_ATTN_ERR_INVALID, "workspace must be 256-byte aligned");
    if (user_ws_bytes < need)
      return fail(SPARSE_ATTN_ERR_INVALID, "workspace holds %zu bytes, this shape needs %zu (sparse_attn_workspace_bytes)",
                  user_ws_bytes, need);
  }
  if (static_scratch && workspace_bytes(s) > kStaticScratchBytes)
    return fail(SPARSE_ATTN_ERR_UNSUPPORTED,
                "this shape needs %zu bytes of scratch, the no-allocation entry point holds %zu "
                "(B*H*Tq*(ceil(Tkv/32)+3)*4 bytes must fit)", workspace_bytes(s), kStaticScratchBytes);

  int dev = 0, cus = 0;
  HIP_TRY(hipGetDevice(&dev));
  if (plan && dev != plan->dev) return fail(SPARSE_ATTN_ERR_INVALID, "the plan was created on device %d, current device is %d", plan->dev, dev);

  PlanBuffers pb;
  if (plan) {
    pb = plan->bufs;
  } else if (use_user_ws) {
    pb = carve((char*)user_ws, s);
  } else if (static_scratch) {
    void* ws = nullptr;
    if (int rc = static_scratch_ptr(&ws)) return rc;
    pb = carve((char*)ws, s);
  } else {
    void* ws = nullptr;
    if (int rc = sa_get_scratch(workspace_bytes(s), stream, &ws)) return rc;
    pb = carve((char*)ws, s);
  }

  HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));

  // Without symbols the blocks are the kernel's business.  Larger query blocks read K and V for more rows at a time; they
  // pay as soon as there are more 128-row blocks than CUs.  24 heads, us, blocks of 64 / 128 / 256 rows: 33024 tokens of
  // 128 channels - / 10850 / 10660, 4608 tokens - / 247 / 230, 9001 tokens 1573 / - / 926, 2000 tokens - / 60 / 55, 1000
  // tokens (192 blocks of 128) - / 24 / 30; 9001 tokens of 64 channels 675 / 547 / 627.  The bits of the result do not
  // depend on the choice: a wave's 32 rows and the order of the keys are the same.
  if (!plan && !cache_flags && !kv_mask && (long long)B * H * ((L + 127) / 128) > cus) {
    bq = D == 128 ? 256 : 128;
    bk = 128;
    s.bq = bq;
    s.bk = bk;
    s.Tq = (L + bq - 1) / bq;
    s.Tkv = (L + bk - 1) / bk;
    s.N = B * H * s.Tq;
    s.row_bytes = (s.Tkv + 7) / 8;
    s.nw32 = (s.Tkv + 31) / 32;
    pb = carve((char*)pb.queues, s);     // (no larger than for the caller's blocks)
  }

  hipEvent_t ev[3] = {nullptr, nullptr, nullptr};
  bool record = timed;
  if (timed) {
    for (auto& e : ev) HIP_TRY(hipEventCreate(&e));
  } else {
    std::lock_guard<std::mutex> lock(g_mu);
    if (g_prof.on && g_prof.calls < g_prof.capacity) {
      for (int t = 0; t < 3; ++t) ev[t] = g_prof.ev[3 * g_prof.calls + t];
      ++g_prof.calls;
      record = true;
    }
  }
  if (record) HIP_TRY(hipEventRecord(ev[0], stream));

  // persistent grid: as many workgroups as the CUs hold (8 waves by registers, 12 with 64 channels; 160 KiB of LDS), fewer if
  // there are fewer items.  With two per CU whatever their size, the 2-wave workgroups of 64-row blocks left half of the
  // waves idle: 9001 tokens, 24 heads of 64, 64 x 128 blocks at 40 % keep: 330 -> 224 us.
  const int keys = attn_keys(D, bq, s.N, plan ? plan->some_cached : cache_flags != nullptr, cus);
  auto room = [&](int mode) -> int {
    const int by_waves = 4 * attn_waves_per_simd(D, mode) / (bq / 32), by_lds = (int)(160 * 1024 / attn_lds(D, bq, keys, mode));
    return cus * (by_waves < by_lds ? by_waves : by_lds);
  };
  // No pre-pass where it cannot help: with no more rows than workgroups the order matters little, and without symbols
  // all rows are equally long, so with up to two per workgroup dealing them out by number does as well.  Every
  // workgroup then decodes its own rows (at most 64 words each).  512 tokens, two heads of 64: 20.1 -> 12.3 us; 4608
  // tokens, 24 heads, dense: 273 -> 261 us.
  // None either where the rows differ and there are between one per CU and two and a quarter per workgroup (counted with two
  // waves on a SIMD): the workgroups sort them.  24 heads, us, queues or dealt / sorted: 4608 tokens, 30 % keep, 56 % cached
  // 56.1 / 50.5; 64 channels, 64-row blocks, 40 % cached 48.4 / 37.2; 6000 tokens (1128 rows on 512 workgroups), 20 % keep
  // 106 / 99, 70 % 312 / 300; 1200 tokens in 64-row blocks (456 rows) 18.0 / 16.3; 16 heads of 777 tokens (208 rows) 12.4 /
  // 13.6.  Beyond, tickets and stealing balance better (7500 tokens, 1416 rows, 40 % keep, 30 % cached 199 / 203; 10500 tokens,
  // 60 % cached 190 / 200), and so they do without a mask, where a row too many for the workgroups of one XCD is a whole row (64
  // channels, 4608 tokens, 40 % cached 127 / 140).  Measured before the last round was turned around (early_of); with it, 60 calls
  // of 39 to 250 rows per XCD, 10 to 90 % keep, up to 90 % cached and both channel counts take 0.67 to 1.002 of the list's time.
  const bool symbols = cache_flags != nullptr || kv_mask != nullptr;
  int mode = kQueues;
  if (!plan && kv_mask && s.nw32 <= kSortWords && s.N > cus && s.N <= kXcds * kSortRows && 4LL * s.N <= 9LL * std::min(room(kSorted), 8 * cus / (bq / 32)))
    mode = kSorted;
  else if (!plan && s.nw32 <= 64 && s.N <= (symbols ? 1 : 2) * room(kDealt))
    mode = kDealt;
  const int grid = s.N < room(mode) ? s.N : room(mode);
  if (!plan && mode == kQueues) {
    if (int rc = launch_plan(cache_flags, kv_mask, s, 1, pb, stream)) return rc;
  }
  if (record) HIP_TRY(hipEventRecord(ev[1], stream));

  AttnParams p;
  p.Q = (const char*)Q;
  p.K = (const char*)K;
  p.V = (const char*)V;
  p.O_cache = (const char*)O_cache;
  p.O = (char*)O;
  p.words = pb.words;
  p.order = pb.order;
  p.queues = pb.queues;
  p.mode = mode;
  p.self_reset = plan != nullptr ? 1 : 0;
  p.raw_flags = cache_flags;
  p.raw_mask = kv_mask;
  p.raw_row_bytes = s.row_bytes;
  p.N = s.N;
  p.BH = B * H;
  p.Tq = s.Tq;
  p.Tkv = s.Tkv;
  p.L = L;
  p.nw32 = s.nw32;
  p.do_copy = (O_cache != nullptr && O_cache != O) ? 1 : 0;
  for (int d = 0; d < kMaxTerms; ++d) p.coef[d] = 0.f;
  for (int d = 0; d + 1 < kMaxTerms; ++d) p.term[d] = nullptr;
  p.n_terms = 0;
  if (fc) {
    p.O_cache = (const char*)fc->terms[0];
    if (fc->n == 1 && fc->coef[0] == 1.0f) {
      p.do_copy = 1;                       // order 0 with weight 1 is the plain copy
    } else {
      p.n_terms = fc->n;
      for (int d = 0; d < fc->n; ++d) p.coef[d] = fc->coef[d];
      for (int d = 1; d < fc->n; ++d) p.term[d - 1] = (const char*)fc->terms[d];
    }
  }
  p.scale_log2 = (float)(1.4426950408889634 / sqrt((double)D));
  int rc = 0;
  if (D == 128 && bq == 256) rc = launch_attn<128, 256, 128>(p, grid, stream);
  else if (D == 128 && bq == 128 && bk == 128) rc = launch_attn<128, 128, 128>(p, grid, stream);
  else if (D == 128 && bq == 128 && bk == 64) rc = launch_attn<128, 128, 64>(p, grid, stream);
  else if (D == 128 && bq == 64 && bk == 128)
    rc = keys == 32 ? launch_attn<128, 64, 128, 32>(p, grid, stream) : launch_attn<128, 64, 128>(p, grid, stream);
  else if (D == 128 && bq == 64 && bk == 64)
    rc = keys == 32 ? launch_attn<128, 64, 64, 32>(p, grid, stream) : launch_attn<128, 64, 64>(p, grid, stream);
  else if (D == 64 && bq == 128 && bk == 128) rc = launch_attn<64, 128, 128>(p, grid, stream);
  else if (D == 64 && bq == 128 && bk == 64) rc = launch_attn<64, 128, 64>(p, grid, stream);
  else if (D == 64 && bq == 64 && bk == 128) rc = launch_attn<64, 64, 128>(p, grid, stream);
  else rc = launch_attn<64, 64, 64>(p, grid, stream);
  if (rc) return rc;

  if (record) HIP_TRY(hipEventRecord(ev[2], stream));
  if (timed) {
    HIP_TRY(hipEventSynchronize(ev[2]));
    float a = 0.f, b = 0.f;
    HIP_TRY(hipEventElapsedTime(&a, ev[0], ev[1]));
    HIP_TRY(hipEventElapsedTime(&b, ev[1], ev[2]));
    if (plan_ms) *plan_ms = a;
    if (attn_ms) *attn_ms = b;
    for (auto& e : ev) HIP_TRY(hipEventDestroy(e));
  }
  return 0;
}

}  // namespace

extern "C" {

int sparse_attn_fwd(const void* Q, const void* K, const void* V, const uint8_t* cache_flags, const uint8_t* kv_mask,
                    const void* O_cache, void* O, int B, int H, int L, int D, int block_q, int block_k) {
  return run(Q, K, V, cache_flags, kv_mask, O_cache, O, B, H, L, D, block_q, block_k, nullptr, nullptr, nullptr,
             false);
}

int sparse_attn_fwd_stream(const void* Q, const void* K, const void* V, const uint8_t* cache_flags,
                           const uint8_t* kv_mask, const void* O_cache, void* O, int B, int H, int L, int D,
                           int block_q, int block_k, void* hip_stream) {
  return run(Q, K, V, cache_flags, kv_mask, O_cache, O, B, H, L, D, block_q, block_k, (hipStream_t)hip_stream,
             nullptr, nullptr, false);
}

int sparse_attn_fwd_timed(const void* Q, const void* K, const void* V, const uint8_t* cache_flags,
                          const uint8_t* kv_mask, const void* O_cache, void* O, int B, int H, int L, int D,
                          int block_q, int block_k, void* hip_stream, float* plan_ms, float* attn_ms) {
  return run(Q, K, V, cache_flags, kv_mask, O_cache, O, B, H, L, D, block_q, block_k, (hipStream_t)hip_stream,
             plan_ms, attn_ms, true);
}

int sparse_attn_fwd_noalloc(const void* Q, const void* K, const void* V, const uint8_t* cache_flags,
                            const uint8_t* kv_mask, const void* O_cache, void* O, int B, int H, int L, int D,
                            int block_q, int block_k, void* hip_stream) {
  return run(Q, K, V, cache_flags, kv_mask, O_cache, O, B, H, L, D, block_q, block_k, (hipStream_t)hip_stream,
             nullptr, nullptr, false, nullptr, nullptr, true);
}

int sparse_attn_fwd_forecast(const void* Q, const void* K, const void* V, const uint8_t* cache_flags,
                             const uint8_t* kv_mask, const void* const* O_terms, const float* coef, int n_terms, void* O,
                             int B, int H, int L, int D, int block_q, int block_k, void* hip_stream) {
  const Forecast fc = {O_terms, coef, n_terms};
  return run(Q, K, V, cache_flags, kv_mask, nullptr, O, B, H, L, D, block_q, block_k, (hipStream_t)hip_stream, nullptr,
             nullptr, false, &fc);
}

int sparse_attn_plan_create(const uint8_t* cache_flags, const uint8_t* kv_mask, int B, int H, int L, int block_q,
                            int block_k, int granularity, void* hip_stream, sparse_attn_plan** plan_out) {
  if (!plan_out) return fail(SPARSE_ATTN_ERR_INVALID, "plan_out must not be NULL");
  *plan_out = nullptr;
  Shape s;
  if (int rc = check_shape(B, H, L, 0, block_q, block_k, false, &s)) return rc;
  if (granularity < 1 || granularity > 64)
    return fail(SPARSE_ATTN_ERR_INVALID, "granularity=%d must be between 1 and 64", granularity);
  sparse_attn_plan* pl = new (std::nothrow) sparse_attn_plan();
  if (!pl) return fail(SPARSE_ATTN_ERR_HIP, "out of host memory");
  pl->s = s;
  pl->gran = granularity;
  pl->some_cached = cache_flags != nullptr;
  pl->mem = nullptr;
  hipError_t e = hipGetDevice(&pl->dev);
  if (e == hipSuccess) e = hipMalloc(&pl->mem, workspace_bytes(s));
  if (e != hipSuccess) {
    delete pl;
    return fail(SPARSE_ATTN_ERR_HIP, "plan allocation failed: %s", hipGetErrorString(e));
  }
  pl->bufs = carve((char*)pl->mem, s);
  if (int rc = launch_plan(cache_flags, kv_mask, s, granularity, pl->bufs, (hipStream_t)hip_stream)) {
    (void)hipFree(pl->mem);
    delete pl;
    return rc;
  }
  *plan_out = pl;
  return 0;
}

int sparse_attn_plan_run(sparse_attn_plan* plan, const void* Q, const void* K, const void* V, const void* O_cache,
                         void* O, int D, void* hip_stream) {
  if (!plan) return fail(SPARSE_ATTN_ERR_INVALID, "plan must not be NULL");
  const Shape& s = plan->s;
  return run(Q, K, V, nullptr, nullptr, O_cache, O, s.B, s.H, s.L, D, s.bq, s.bk, (hipStream_t)hip_stream, nullptr,
             nullptr, false, nullptr, plan);
}

int sparse_attn_plan_run_forecast(sparse_attn_plan* plan, const void* Q, const void* K, const void* V,
                                  const void* const* O_terms, const float* coef, int n_terms, void* O, int D,
                                  void* hip_stream) {
  if (!plan) return fail(SPARSE_ATTN_ERR_INVALID, "plan must not be NULL");
  const Shape& s = plan->s;
  const Forecast fc = {O_terms, coef, n_terms};
  return run(Q, K, V, nullptr, nullptr, nullptr, O, s.B, s.H, s.L, D, s.bq, s.bk, (hipStream_t)hip_stream, nullptr,
             nullptr, false, &fc, plan);
}

int sparse_attn_plan_destroy(sparse_attn_plan* plan) {
  if (!plan) return 0;
  const hipError_t e = hipFree(plan->mem);     // waits for work that still uses the buffer
  delete plan;
  if (e != hipSuccess) return fail(SPARSE_ATTN_ERR_HIP, "hipFree failed: %s", hipGetErrorString(e));
  return 0;
}

int sparse_attn_fwd_workspace(const void* Q, const void* K, const void* V, const uint8_t* cache_flags,
                              const uint8_t* kv_mask, const void* O_cache, void* O, int B, int H, int L, int D,
                              int block_q, int block_k, void* workspace, size_t workspace_size, void* hip_stream) {
  return run(Q, K, V, cache_flags, kv_mask, O_cache, O, B, H, L, D, block_q, block_k, (hipStream_t)hip_stream, nullptr,
             nullptr, false, nullptr, nullptr, false, workspace, workspace_size, true);
}

int sparse_attn_release_scratch(void* hip_stream) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  void* ptr = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_mu);
    auto it = g_scratch.find(std::make_pair(dev, hip_stream));
    if (it == g_scratch.end()) return 0;
    ptr = it->second.ptr;
    g_scratch.erase(it);
  }
  if (ptr) {
    HIP_TRY(hipStreamSynchronize((hipStream_t)hip_stream));    // work that still uses the buffer
    HIP_TRY(hipFree(ptr));
  }
  return 0;
}

size_t sparse_attn_workspace_bytes(int B, int H, int L, int block_q, int block_k) {
  Shape s;
  if (check_shape(B, H, L, 0, block_q, block_k, false, &s)) return 0;
  return workspace_bytes(s);
}

int sparse_attn_count_kept(const uint8_t* cache_flags, const uint8_t* kv_mask, int B, int H, int L, int block_q,
                           int block_k, unsigned long long* kept_pairs, unsigned long long* total_pairs) {
  Shape s;
  if (int rc = check_shape(B, H, L, 0, block_q, block_k, false, &s)) return rc;
  if (!kept_pairs) return fail(SPARSE_ATTN_ERR_INVALID, "kept_pairs must not be NULL");
  unsigned long long kept = 0;
  for (int row = 0; row < s.N; ++row) {
    if (cache_flags && cache_flags[row]) continue;
    if (!kv_mask) {
      kept += (unsigned long long)s.Tkv;
      continue;
    }
    const uint8_t* r = kv_mask + (size_t)row * s.row_bytes;
    for (int byte = 0; byte < s.row_bytes; ++byte) {
      unsigned v = r[byte];
      const int valid = s.Tkv - 8 * byte;
      if (valid < 8) v &= (0xffu << (8 - valid)) & 0xffu;
      kept += (unsigned long long)__builtin_popcount(v);
    }
  }
  *kept_pairs = kept;
  if (total_pairs) *total_pairs = (unsigned long long)s.N * (unsigned long long)s.Tkv;
  return 0;
}

int sparse_attn_pack_mask(const uint8_t* logical, long long rows, int Tkv, uint8_t* packed) {
  if (!logical || !packed || rows < 0 || Tkv <= 0)
    return fail(SPARSE_ATTN_ERR_INVALID, "pack_mask: bad arguments (rows=%lld Tkv=%d)", rows, Tkv);
  const int row_bytes = (Tkv + 7) / 8;
  for (long long r = 0; r < rows; ++r) {
    const uint8_t* src = logical + (size_t)r * Tkv;
    uint8_t* dst = packed + (size_t)r * row_bytes;
    for (int byte = 0; byte < row_bytes; ++byte) {
      unsigned v = 0;
      for (int t = 0; t < 8; ++t) {
        const int j = 8 * byte + t;
        if (j < Tkv && src[j]) v |= 0x80u >> t;
      }
      dst[byte] = (uint8_t)v;
    }
  }
  return 0;
}

int sparse_attn_profile_begin(int max_calls) {
  if (max_calls <= 0 || max_calls > (1 << 20)) return fail(SPARSE_ATTN_ERR_INVALID, "profile_begin: bad max_calls %d", max_calls);
  std::lock_guard<std::mutex> lock(g_mu);
  if (g_prof.on) return fail(SPARSE_ATTN_ERR_INVALID, "profile_begin: a profile is already open");
  g_prof.ev = new hipEvent_t[3 * (size_t)max_calls];
  for (int t = 0; t < 3 * max_calls; ++t) {
    hipError_t e = hipEventCreate(&g_prof.ev[t]);
    if (e != hipSuccess) {
      for (int u = 0; u < t; ++u) (void)hipEventDestroy(g_prof.ev[u]);
      delete[] g_prof.ev;
      g_prof.ev = nullptr;
      return fail(SPARSE_ATTN_ERR_HIP, "hipEventCreate failed: %s", hipGetErrorString(e));
    }
  }
  g_prof.capacity = max_calls;
  g_prof.calls = 0;
  g_prof.on = true;
  return 0;
}

int sparse_attn_profile_end(int* calls, double* plan_ms_total, double* attn_ms_total) {
  std::lock_guard<std::mutex> lock(g_mu);
  if (!g_prof.on) return fail(SPARSE_ATTN_ERR_INVALID, "profile_end: no profile is open");
  int rc = 0;
  double plan = 0.0, attn = 0.0;
  for (int c = 0; c < g_prof.calls && rc == 0; ++c) {
    hipError_t e = hipEventSynchronize(g_prof.ev[3 * c + 2]);
    float a = 0.f, b = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&a, g_prof.ev[3 * c], g_prof.ev[3 * c + 1]);
    if (e == hipSuccess) e = hipEventElapsedTime(&b, g_prof.ev[3 * c + 1], g_prof.ev[3 * c + 2]);
    if (e != hipSuccess) rc = fail(SPARSE_ATTN_ERR_HIP, "profile_end: %s", hipGetErrorString(e));
    plan += a;
    attn += b;
  }
  for (int t = 0; t < 3 * g_prof.capacity; ++t) (void)hipEventDestroy(g_prof.ev[t]);
  delete[] g_prof.ev;
  if (calls) *calls = g_prof.calls;
  if (plan_ms_total) *plan_ms_total = plan;
  if (attn_ms_total) *attn_ms_total = attn;
  g_prof = Profile();
  return rc;
}


const char* sparse_attn_last_error(void) { return g_err; }

int sparse_attn_version(void) { return 100; }

}  // extern "C"
