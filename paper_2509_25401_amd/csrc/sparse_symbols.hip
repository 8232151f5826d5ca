// Sparse-symbol generation of an Update step (Section 3.3 "Logical Masks Generation", Equation 1, and
// the tau_kv / S_q rules of the settings table in the appendix) for gfx950.
//
// Three kernels, all in fp32 (vector instructions, and matrix instructions for the map's scores):
//   pool_blocks   mean of the n*b_q query rows / n*b_k key rows of every pooled block (granularity n): the only
//                 pass over Q and K, HBM-bound (reads both tensors once, 16 bytes per lane, row-contiguous)
//   map_rows      one workgroup per 16 rows of the compressed attention map of one head: scores of the
//                 pooled queries against all pooled keys (scale 1/sqrt(d)), row softmax, then for
//                 every row the block-skipping rule -- a key block is skipped iff the sum of all row
//                 entries that come at or before it in ascending order (ties by index) stays <= tau_kv
//                 -- packed most-significant-bit first into the kv_mask row.  The text rows and text
//                 columns of the map (all that the caching rule needs) go to scratch memory.
//   select_blocks one workgroup per head: contribution C_u = sum over text rows of their weight on
//                 vision key block u (carried over to the vision query blocks by token overlap when
//                 n*b_q != n*b_k), guidance G_v = sum over text columns of the softmax, along the vision
//                 axis, of the vision rows' weights on that column; Equation 1 caches v iff its
//                 ascending cumulative sums of C and of G both stay <= tau_c times the totals; text
//                 blocks are never cached; if the share of blocks left to compute drops below S_q,
//                 every block of the head is cached.
// Neither rule needs a sort: both select everything up to a threshold value, found by bisection on the bits of that
// value.  At 33024 tokens and 24 heads pool_blocks is at the memory's rate (61 us, 6.6 TB/s), the other two (24 and 8) are
// latency.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "sparse_attn.h"
#include "sparse_attn_internal.h"

namespace {

// Map rows per workgroup, 16 lanes to a row in four waves; rows of more than 512 entries lie in LDS, two to a wave.  The time is
// the chain of one workgroup, and two of them on a CU overlap scores of the one with the search of the other (32 rows and
// eight waves, the call, us: 24 heads of 118 blocks 50.5 / 46.5, 13 heads of 141 39.6 / 34.6, 5 heads of 469 75.5 / 67.9, 24 heads
// of 258 92.9 / 92.9).
constexpr int kMapRows = 16;
constexpr int map_threads(int np) { return np > 0 ? 256 : 512; }
constexpr int kMaxBlocks = 2048;     // blocks per sequence the LDS arrays are sized for

// Sum over the 64 lanes, the same bits in every lane, without going through LDS: exchanges inside a row of 16
// lanes are DPP operands of the add, the two exchanges between rows are the gfx950 lane-swap instructions.
// Every step adds a value and its mirror partner's, so both partners compute the same sum.
__device__ __forceinline__ float wave_sum_dpp(float v) {
  auto dpp = [](float x, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  v += dpp(v, std::integral_constant<int, 0xB1>{});    // quad_perm [1,0,3,2]: lane ^ 1
  v += dpp(v, std::integral_constant<int, 0x4E>{});    // quad_perm [2,3,0,1]: lane ^ 2
  v += dpp(v, std::integral_constant<int, 0x141>{});   // row_half_mirror: the other quad of each 8 lanes
  v += dpp(v, std::integral_constant<int, 0x140>{});   // row_mirror: the other 8 lanes of each row
  {
    const unsigned bits = __float_as_uint(v);
    const auto sw = __builtin_amdgcn_permlane16_swap(bits, bits, false, false);   // rows 0<->1, 2<->3
    v = __uint_as_float((unsigned)sw[0]) + __uint_as_float((unsigned)sw[1]);
  }
  {
    const unsigned bits = __float_as_uint(v);
    const auto sw = __builtin_amdgcn_permlane32_swap(bits, bits, false, false);   // lanes 0-31 <-> 32-63
    v = __uint_as_float((unsigned)sw[0]) + __uint_as_float((unsigned)sw[1]);
  }
  return v;
}

// Pooled queries [BH][Tq][D], then pooled keys [BH][Tk][D]: mean over the pooled block's rows.  Grid
// (BH * max(Tq, Tk), 2), y = 0 for Q (pool_q rows per block), 1 for K (pool_k rows per block).
template <int D>
__global__ void __launch_bounds__(256) pool_blocks(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
                                                   float* __restrict__ pooled, int pool_q, int pool_k, int Tq, int Tk,
                                                   int L, long long n_q_blocks) {
  constexpr int TPR = D / 8;          // threads per row, 8 bf16 = 16 bytes each
  constexpr int RPP = 256 / TPR;      // rows per pass
  __shared__ float part[RPP][D];
  const int Tmax = max(Tq, Tk);
  const int T = blockIdx.y ? Tk : Tq, pool = blockIdx.y ? pool_k : pool_q;
  // pooled block t of head bh; the last block of a head may be short: the mean is over the rows that exist
  const int bh = blockIdx.x / Tmax, t = blockIdx.x - bh * Tmax;
  if (t >= T) return;
  const int rows = min(pool, L - t * pool);
  const uint16_t* src = (blockIdx.y ? K : Q) + ((size_t)bh * L + (size_t)t * pool) * D;
  const int c = threadIdx.x % TPR, r0 = threadIdx.x / TPR;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int r = r0; r < rows; r += RPP) {
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
    const u32x4 v = __builtin_nontemporal_load((const u32x4*)(src + (size_t)r * D + c * 8));   // read once
    const unsigned w[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc[2 * e] += __uint_as_float(w[e] << 16);
      acc[2 * e + 1] += __uint_as_float(w[e] & 0xffff0000u);
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) part[r0][c * 8 + e] = acc[e];
  __syncthreads();
  if (threadIdx.x < D) {
    float s = 0.f;
    for (int r = 0; r < RPP; ++r) s += part[r][threadIdx.x];
    const size_t slot = (blockIdx.y ? (size_t)n_q_blocks : 0) + (size_t)bh * T + t;
    pooled[slot * D + threadIdx.x] = s / (float)rows;
  }
}

// Maximum over the 64 lanes, the same exchanges.
__device__ __forceinline__ float wave_max_dpp(float v) {
  auto dpp = [](float x, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  v = fmaxf(v, dpp(v, std::integral_constant<int, 0xB1>{}));
  v = fmaxf(v, dpp(v, std::integral_constant<int, 0x4E>{}));
  v = fmaxf(v, dpp(v, std::integral_constant<int, 0x141>{}));
  v = fmaxf(v, dpp(v, std::integral_constant<int, 0x140>{}));
  {
    const unsigned bits = __float_as_uint(v);
    const auto sw = __builtin_amdgcn_permlane16_swap(bits, bits, false, false);
    v = fmaxf(__uint_as_float((unsigned)sw[0]), __uint_as_float((unsigned)sw[1]));
  }
  {
    const unsigned bits = __float_as_uint(v);
    const auto sw = __builtin_amdgcn_permlane32_swap(bits, bits, false, false);
    v = fmaxf(__uint_as_float((unsigned)sw[0]), __uint_as_float((unsigned)sw[1]));
  }
  return v;
}

// The first steps of the above: over the 16 lanes of a row of lanes.
template <class Op>
__device__ __forceinline__ float row16_reduce(float v, Op op) {
  auto dpp = [](float x, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  v = op(v, dpp(v, std::integral_constant<int, 0xB1>{}));
  v = op(v, dpp(v, std::integral_constant<int, 0x4E>{}));
  v = op(v, dpp(v, std::integral_constant<int, 0x141>{}));
  return op(v, dpp(v, std::integral_constant<int, 0x140>{}));
}
template <int G>
__device__ __forceinline__ float group_sum(float v) {
  if constexpr (G == 64) return wave_sum_dpp(v);
  else return row16_reduce(v, [](float a, float b) { return a + b; });
}
template <int G>
__device__ __forceinline__ float group_max(float v) {
  if constexpr (G == 64) return wave_max_dpp(v);
  else return row16_reduce(v, [](float a, float b) { return fmaxf(a, b); });
}

// G lanes (a wave, or 16 lanes: four rows per wave) hold one row of values, entry l + G * n in the n-th place of lane l:
// NP > 0: in registers (those past T hold +inf, which no finite threshold admits), NP = 0: in LDS.
template <int G, int NP>
struct Row {
  float v[NP > 0 ? NP : 1];
  const float* lds;
  int T, l;
  __device__ __forceinline__ void load(const float* p, int T_, int l_) {
    lds = p;
    T = T_;
    l = l_;
    if constexpr (NP > 0) {
#pragma unroll
      for (int n = 0; n < NP; ++n) v[n] = l + G * n < T ? p[l + G * n] : INFINITY;
    }
  }
  template <class F>
  __device__ __forceinline__ void each(F&& f) const {
    if constexpr (NP > 0) {
#pragma unroll
      for (int n = 0; n < NP; ++n) f(n, v[n]);
    } else {
      for (int n = 0; G * n < T; ++n) f(n, l + G * n < T ? lds[l + G * n] : INFINITY);
    }
  }
  // sum of the entries <= x, the same bits in every lane of the row
  __device__ __forceinline__ float sum_upto(float x) const {
    float s = 0.f;
    each([&](int, float a) { s += a <= x ? a : 0.f; });
    return group_sum<G>(s);
  }
};

// Selection of a prefix of the ascending order without a sort.  "Select entry j iff the ascending cumulative sum at j is
// <= limit" selects all entries up to some value theta (plus, among entries equal to the next value, the first few in
// index order).  S(x) = sum of the entries <= x is a non-decreasing step function of x (also as computed here in
// fp32: a fixed summation structure is monotone in every term), so the largest float theta with S(theta) <= limit is
// found by fixing its bits from the top: at most 31 conditional sums per row instead of one per entry.  The lower bits
// are not needed once there is at most one entry among the candidates left: one more sum says whether it is admitted
// (looked at every third bit; mostly after some 17 bits of 31: the call at 33024 tokens and 24 heads 104.7 -> 98.3 us, 1300 tokens
// and 7 heads 21.6 -> 16.8).
// Candidates below the smallest entry have the sum 0 and those from the largest on the sum of all: where that holds for
// every row of the wave nothing is added up (the upper exponent bits of a softmax: 98.6 -> 94.8 us).
// M rows per group of lanes are searched together so that their reductions overlap.  sum[r] returns S(theta[r]).
template <int G, int NP, int M>
__device__ __forceinline__ void find_thresholds(const Row<G, NP> (&row)[M], const float (&limit)[M], float (&theta)[M], float (&sum)[M]) {
  unsigned lo[M];
  float least[M], most[M], all[M];
#pragma unroll
  for (int r = 0; r < M; ++r) {
    lo[r] = 0u;
    sum[r] = 0.f;
    least[r] = all[r] = 0.f;
    most[r] = INFINITY;
    if constexpr (NP > 0) {            // (from LDS these passes cost more than the sums they save)
      least[r] = INFINITY;
      most[r] = -INFINITY;
      row[r].each([&](int, float a) {
        least[r] = fminf(least[r], a);
        most[r] = fmaxf(most[r], a < INFINITY ? a : -INFINITY);
      });
      least[r] = -group_max<G>(-least[r]);
      most[r] = group_max<G>(most[r]);
      all[r] = row[r].sum_upto(most[r]);
    }
  }
  for (int bit = 30; bit >= 0; --bit) {
    float s[M];
    bool known = true;
#pragma unroll
    for (int r = 0; r < M; ++r) {
      const float x = __uint_as_float(lo[r] | (1u << bit));
      s[r] = x < least[r] ? 0.f : all[r];
      known = known && (x < least[r] || x >= most[r]);
    }
    if (__builtin_amdgcn_ballot_w64(!known) != 0ull) {
#pragma unroll
      for (int r = 0; r < M; ++r) s[r] = row[r].sum_upto(__uint_as_float(lo[r] | (1u << bit)));
    }
#pragma unroll
    for (int r = 0; r < M; ++r) {
      // (the pattern of +inf and those above it are no candidates)
      if (s[r] <= limit[r] && (lo[r] | (1u << bit)) < 0x7f800000u) {
        lo[r] |= 1u << bit;
        sum[r] = s[r];
      }
    }
    if (bit % 3 == 2 && bit <= 17 && bit > 2) {
      bool open = false;
#pragma unroll
      for (int r = 0; r < M; ++r) {
        // entries above lo and up to lo | the bits below (patterns of positive numbers are ordered like the numbers)
        int inside = 0;
        row[r].each([&](int, float a) { inside += __float_as_uint(a) - lo[r] - 1u < (1u << bit) - 1u ? 1 : 0; });
        open |= group_sum<G>((float)inside) > 1.f;
      }
      if (__builtin_amdgcn_ballot_w64(open) == 0ull) {
#pragma unroll
        for (int r = 0; r < M; ++r) {
          const unsigned to = lo[r] | ((1u << bit) - 1u);
          const float s_to = row[r].sum_upto(__uint_as_float(to));
          if (s_to <= limit[r]) {
            lo[r] = to;
            sum[r] = s_to;
          }
        }
        break;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < M; ++r) theta[r] = limit[r] >= 0.f ? __uint_as_float(lo[r]) : -1.f;   // (a limit that is no number admits nothing)
}

// This row's bits of a wave ballot.
template <int G>
__device__ __forceinline__ unsigned long long group_bits(unsigned long long ballot, int lane) {
  return G == 64 ? ballot : (ballot >> (lane & 48)) & 0xffffull;
}

// Entries equal to the smallest value above theta come next in the ascending order, in index order: how many of
// them still fit under the limit when added one by one to S(theta).  (With distinct values: none, by the choice of theta.)
template <int G, int NP>
__device__ __forceinline__ void next_value_ties(const Row<G, NP>& row, int lane, float theta, float s_theta, float limit,
                                                float& next, int& n_more) {
  float nx = INFINITY;
  row.each([&](int, float a) { nx = fminf(nx, a > theta ? a : INFINITY); });
  nx = -group_max<G>(-nx);
  int m = 0;
  row.each([&](int, float a) { m += __popcll(group_bits<G>(__ballot(a == nx && a < INFINITY), lane)); });
  int k = 0;
  float run = s_theta;
  while (k < m) {
    run += nx;
    if (!(run <= limit)) break;
    ++k;
  }
  next = nx;
  n_more = k;
}

// 16 rows of one head's map per workgroup.
//   scores    fp32 matrix instructions, 16 x 16 tiles with 4 products a step: lane (r = lane % 16, g = lane / 16) of an
//             operand holds channels 16 * u + 4 * g + e of row r, so that both operands come straight from the pooled
//             means with 16-byte loads of which four lanes share a line, and step (u, e) adds the four channels with
//             that e.  The waves take the tiles of 16 keys in turn; the keys of the next two tiles are on their way.
//   softmax, skipping rule: 16 lanes per row, four rows per wave, in registers (NP entries per lane); a row per wave and
//             two rows one after the other from LDS where NP = 0.  (The search is issue bound: with a row per wave half
//             of its instructions were the reduction over 64 lanes.)
// Dot products with both operands from LDS and the search over 64 lanes took 50 us at 33024 tokens and 24 heads, matrix
// instructions and 16 lanes 30, this 24.
// Dynamic LDS: map rows [kMapRows][T_pad].
template <int D, int NP>
__global__ void __launch_bounds__(map_threads(NP)) map_rows(const float* __restrict__ pooled, long long n_q_blocks, int Tq, int T, int T_pad,
                                                               int n_tq, int n_t, int row_bytes, float scale, float tau_kv,
                                                               uint8_t* __restrict__ kv_mask, float* __restrict__ text_rows,
                                                               float* __restrict__ text_cols) {
  extern __shared__ float p[];
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  constexpr int NWAVES = map_threads(NP) / 64;
  const int tid = threadIdx.x, w = tid / 64, lane = tid % 64;
  // T = pooled key blocks (columns of the map), n_t of them text; Tq = pooled query blocks (rows), n_tq of them text
  const int groups = (Tq + kMapRows - 1) / kMapRows;
  // The workgroups of a head run on one XCD (workgroup n on XCD n mod 8) and find its pooled keys in that L2 (the call 94.3 ->
  // 93.0 us); heads past a multiple of eight are spread.
  const int heads = (int)(gridDim.x / groups), whole = heads / 8 * 8;
  int bh, i0;
  if ((int)blockIdx.x < whole * groups) {
    const int at = blockIdx.x / 8;
    bh = (int)(blockIdx.x % 8) + 8 * (at / groups);
    i0 = at % groups * kMapRows;
  } else {
    bh = blockIdx.x / groups;
    i0 = (blockIdx.x % groups) * kMapRows;
  }
  const float* qt = pooled + (size_t)bh * Tq * D;
  const float* kt = pooled + ((size_t)n_q_blocks + (size_t)bh * T) * D;
  const int r16 = lane & 15, g = lane >> 4;

  constexpr int V = D / 16;                       // 16-byte pieces of a lane's channels
  auto fetch = [&](const float* base, int row, f32x4 (&v)[V]) {
    const f32x4* src = (const f32x4*)(base + (size_t)row * D) + g;
#pragma unroll
    for (int u = 0; u < V; ++u) v[u] = src[4 * u];
  };
  f32x4 q[V], k[3][V];
  const int tiles = (T + 15) / 16;
  auto fetch_tile = [&](int t, f32x4 (&v)[V]) { fetch(kt, min(16 * min(t, tiles - 1) + r16, T - 1), v); };
  fetch_tile(w, k[0]);
  fetch(qt, min(i0 + r16, Tq - 1), q);            // rows past the end repeat the last one
  constexpr bool kFew = NP == 2 || NP == 4;       // at most four tiles of keys: one per wave, nothing to fetch ahead
  if constexpr (!kFew) fetch_tile(w + NWAVES, k[1]);
  for (int t = w; t < tiles; t += NWAVES) {
    if constexpr (!kFew) fetch_tile(t + 2 * NWAVES, k[2]);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < V; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(q[u][e], k[0][u][e], acc, 0, 0, 0);
    const int j = 16 * t + r16;                   // accumulator: column lane % 16, rows 4 * (lane / 16) + 0..3
    if (j < T) {
#pragma unroll
      for (int e = 0; e < 4; ++e) p[(4 * g + e) * T_pad + j] = acc[e] * scale;
    }
    if constexpr (!kFew) {
#pragma unroll
      for (int u = 0; u < V; ++u) {
        k[0][u] = k[1][u];
        k[1][u] = k[2][u];
      }
    }
  }
  __syncthreads();

  auto export_text = [&](int i, int j, float v) {
    if (i < n_tq) text_rows[((size_t)bh * n_tq + i) * T + j] = v;         // i < n_tq < Tq
    if (j < n_t && i < Tq) text_cols[((size_t)bh * Tq + i) * n_t + j] = v;
  };
  const float limit[1] = {tau_kv};
  float theta[1], s_theta[1], next;
  int n_more, seen = 0;                           // seen: entries equal to `next` at smaller indices
  if constexpr (NP > 0) {
    const int i = i0 + 4 * w + g;                 // this lane's row
    Row<16, NP> row[1];
    row[0].load(p + (4 * w + g) * T_pad, T, r16);
    auto& v = row[0].v;
    float m = -INFINITY, sum = 0.f;
#pragma unroll
    for (int n = 0; n < NP; ++n) m = fmaxf(m, r16 + 16 * n < T ? v[n] : -INFINITY);
    m = group_max<16>(m);
#pragma unroll
    for (int n = 0; n < NP; ++n) {
      v[n] = r16 + 16 * n < T ? expf(v[n] - m) : 0.f;
      sum += v[n];
    }
    sum = group_sum<16>(sum);
#pragma unroll
    for (int n = 0; n < NP; ++n) {
      const int j = r16 + 16 * n;
      v[n] = j < T ? v[n] / sum : INFINITY;
      if (j < T) export_text(i, j, v[n]);
    }
    find_thresholds<16, NP, 1>(row, limit, theta, s_theta);
    next_value_ties(row[0], lane, theta[0], s_theta[0], tau_kv, next, n_more);
    const unsigned long long below = (1ull << r16) - 1ull;
#pragma unroll
    for (int n = 0; n < NP; ++n) {
      const unsigned long long tie = group_bits<16>(__ballot(v[n] == next), lane);
      const bool skip = v[n] <= theta[0] || (v[n] == next && seen + __popcll(tie & below) < n_more);
      seen += __popcll(tie);
      const unsigned kept = (unsigned)group_bits<16>(__ballot(r16 + 16 * n < T && !skip), lane);   // bit b = block 16 * n + b
      // the row's first two lanes write two bytes; first block of a byte = bit 7
      const int byte = 2 * n + r16;
      if (r16 < 2 && i < Tq && byte < row_bytes)
        kv_mask[((size_t)bh * Tq + i) * row_bytes + byte] = (uint8_t)(__brev((kept >> (8 * r16)) & 0xffu) >> 24);
    }
  } else {
    for (int rr = 0; rr < 2; ++rr) {
      const int i = i0 + 2 * w + rr;
      float* pr = p + (2 * w + rr) * T_pad;
      float m = -INFINITY, sum = 0.f;
      for (int j = lane; j < T; j += 64) m = fmaxf(m, pr[j]);
      m = wave_max_dpp(m);
      for (int j = lane; j < T; j += 64) {
        const float e = expf(pr[j] - m);
        pr[j] = e;
        sum += e;
      }
      sum = wave_sum_dpp(sum);
      for (int j = lane; j < T; j += 64) {
        const float v = pr[j] / sum;
        pr[j] = v;
        export_text(i, j, v);
      }
      Row<64, 0> row[1];
      row[0].load(pr, T, lane);                   // (a lane reads what it wrote itself)
      find_thresholds<64, 0, 1>(row, limit, theta, s_theta);
      next_value_ties(row[0], lane, theta[0], s_theta[0], tau_kv, next, n_more);
      const unsigned long long below = (1ull << lane) - 1ull;
      seen = 0;
      row[0].each([&](int n, float a) {
        const unsigned long long tie = __ballot(a == next);
        const bool skip = a <= theta[0] || (a == next && seen + __popcll(tie & below) < n_more);
        seen += __popcll(tie);
        const unsigned long long kept = __ballot(lane + 64 * n < T && !skip);      // bit b = block 64 * n + b
        const int byte = 8 * n + lane;
        if (lane < 8 && i < Tq && byte < row_bytes)
          kv_mask[((size_t)bh * Tq + i) * row_bytes + byte] = (uint8_t)(__brev((unsigned)(kept >> (8 * lane)) & 0xffu) >> 24);
      });
    }
  }
}

// One workgroup per head.  Tq / Tk pooled query / key blocks, n_tq / n_tk of them text; pool_q / pool_k tokens per pooled
// block.  Waves take the text columns side by side for G, then wave 0 searches the threshold of C and wave 1 that of
// G (19 us with a sum over all entries per entry, 33024 tokens; with the search 12, now 8).
template <int NP>
__global__ void __launch_bounds__(256) select_blocks(const float* __restrict__ text_rows,
                                                     const float* __restrict__ text_cols, int Tq, int Tk, int n_tq,
                                                     int n_tk, int pool_q, int pool_k, int L, float tau_c, float s_q,
                                                     uint8_t* __restrict__ cache_flags) {
  __shared__ float CG[2][kMaxBlocks], Ck[kMaxBlocks], E[4][kMaxBlocks];
  __shared__ float theta_s[2], next_s[2];
  __shared__ int more_s[2];
  __shared__ int cached_s;
  const int bh = blockIdx.x, Tv = Tq - n_tq, Tu = Tk - n_tk, tid = threadIdx.x;
  const int w = tid / 64, lane = tid % 64;
  const float* tr = text_rows + (size_t)bh * n_tq * Tk;
  const float* tc = text_cols + (size_t)bh * Tq * n_tk;
  if (tid == 0) cached_s = 0;
  // contribution of every vision key block: what the text rows put on it
  for (int u = tid; u < Tu; u += 256) {
    float c = 0.f;
    for (int j = 0; j < n_tq; ++j) c += tr[(size_t)j * Tk + n_tk + u];
    Ck[u] = c;
  }
  for (int v = tid; v < Tv; v += 256) CG[1][v] = 0.f;
  for (int j0 = 0; j0 < n_tk; j0 += 4) {
    const int j = j0 + w;
    if (j < n_tk) {
      float m = -INFINITY, s = 0.f;
      if constexpr (NP > 0) {
        // in registers, all loads under way at once (entry by entry through LDS the call took 0.8 us longer)
        float x[NP];
#pragma unroll
        for (int n = 0; n < NP; ++n) x[n] = lane + 64 * n < Tv ? tc[(size_t)(n_tq + lane + 64 * n) * n_tk + j] : -INFINITY;
#pragma unroll
        for (int n = 0; n < NP; ++n) m = fmaxf(m, x[n]);
        m = wave_max_dpp(m);
#pragma unroll
        for (int n = 0; n < NP; ++n) {
          x[n] = lane + 64 * n < Tv ? expf(x[n] - m) : 0.f;
          s += x[n];
        }
        s = wave_sum_dpp(s);
#pragma unroll
        for (int n = 0; n < NP; ++n)
          if (lane + 64 * n < Tv) E[w][lane + 64 * n] = x[n] / s;
      } else {
        for (int v = lane; v < Tv; v += 64) {
          const float x = tc[(size_t)(n_tq + v) * n_tk + j];
          E[w][v] = x;
          m = fmaxf(m, x);
        }
        m = wave_max_dpp(m);
        for (int v = lane; v < Tv; v += 64) {
          const float e = expf(E[w][v] - m);
          E[w][v] = e;
          s += e;
        }
        s = wave_sum_dpp(s);
        for (int v = lane; v < Tv; v += 64) E[w][v] /= s;
      }
    }
    __syncthreads();
    for (int v = tid; v < Tv; v += 256)
      for (int jj = 0; jj < min(4, n_tk - j0); ++jj) CG[1][v] += E[jj][v];   // in column order; v belongs to one thread
    __syncthreads();
  }
  for (int v = tid; v < Tv; v += 256) {
    float c;
    if (pool_q == pool_k) {
      c = Ck[v];
    } else {
      // carried over to the query axis: every key block's contribution spread evenly over its tokens
      c = 0.f;
      const int q0 = (n_tq + v) * pool_q, q1 = min(q0 + pool_q, L);
      const int u_lo = max(q0 / pool_k - n_tk, 0), u_hi = min((q1 - 1) / pool_k - n_tk, Tu - 1);
      for (int u = u_lo; u <= u_hi; ++u) {
        const int k0 = (n_tk + u) * pool_k, k1 = min(k0 + pool_k, L);
        const int common = min(k1, q1) - max(k0, q0);
        if (common > 0) c += Ck[u] * (float)common / (float)(k1 - k0);
      }
    }
    CG[0][v] = c;
  }
  __syncthreads();
  if (w < 2) {
    // the total is the sum of everything in the same summation structure: tau_c = 1 then admits every block
    Row<64, NP> row[1];
    row[0].load(CG[w], Tv, lane);
    float all = 0.f;
    for (int v = lane; v < Tv; v += 64) all += CG[w][v];
    all = wave_sum_dpp(all);
    const float limit[1] = {tau_c * all};
    float theta[1], s_theta[1], next;
    int n_more;
    find_thresholds<64, NP, 1>(row, limit, theta, s_theta);
    next_value_ties(row[0], lane, theta[0], s_theta[0], limit[0], next, n_more);
    if (lane == 0) {
      theta_s[w] = theta[0];
      next_s[w] = next;
      more_s[w] = n_more;
    }
  }
  __syncthreads();
  // decisions: 64 blocks per wave and round; equal entries are admitted in index order, so their ranks need the
  // entries before them (ties are rare: counted only where some are admitted)
  uint8_t* out = cache_flags + (size_t)bh * Tq;
  auto admitted = [&](int which, int v) -> bool {
    const float x = CG[which][v];
    if (x <= theta_s[which]) return true;
    if (more_s[which] == 0 || x != next_s[which]) return false;
    int before = 0;
    for (int u = 0; u < v; ++u) before += CG[which][u] == x ? 1 : 0;
    return before < more_s[which];
  };
  int n_cached = 0;
  unsigned mine = 0;                               // decisions of this thread's blocks, bit n = block tid + 256 n
  for (int v = tid, n = 0; v < Tv; v += 256, ++n) {
    const bool cached = admitted(0, v) && admitted(1, v);
    mine |= (cached ? 1u : 0u) << n;
    n_cached += cached ? 1 : 0;
  }
  for (int o = 32; o > 0; o >>= 1) n_cached += __shfl_xor(n_cached, o);
  if (lane == 0) atomicAdd(&cached_s, n_cached);
  __syncthreads();
  const bool degrade = ((float)Tq - (float)cached_s) / (float)Tq < s_q;      // counts stay far below 2^24
  for (int b = tid; b < n_tq; b += 256) out[b] = degrade ? 1 : 0;
  for (int v = tid, n = 0; v < Tv; v += 256, ++n) out[n_tq + v] = (degrade || ((mine >> n) & 1u)) ? 1 : 0;
}

// Entries per lane, 16 lanes to a row: powers of two, and 17 because 33024 tokens in blocks of 128 are 258 blocks, which
// would fall into the tier of 512.  A tier costs what its last size costs (24 heads, blocks of 64 tokens, us: 258 entries
// 64, with 32 registers 71; 273 entries, the first in that tier, 74: 32 registers a lane, 76 scalar registers spilled).
int map_np(int T) { return T <= 32 ? 2 : T <= 64 ? 4 : T <= 128 ? 8 : T <= 272 ? 17 : T <= 512 ? 32 : 0; }
template <int D>
auto map_for(int T) {
  switch (map_np(T)) {
    case 2: return map_rows<D, 2>;
    case 4: return map_rows<D, 4>;
    case 8: return map_rows<D, 8>;
    case 17: return map_rows<D, 17>;
    case 32: return map_rows<D, 32>;
    default: return map_rows<D, 0>;
  }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

#define HIP_TRY(expr)                                                                                \
  do {                                                                                               \
    hipError_t e_ = (expr);                                                                          \
    if (e_ != hipSuccess) return sa_fail(SPARSE_ATTN_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

}  // namespace

extern "C" {

int sparse_symbols_update_granular(const void* Q, const void* K, uint8_t* cache_flags, uint8_t* kv_mask, int B, int H,
                                   int L, int D, int block_q, int block_k, int granularity, int text_tokens, float tau_c,
                                   float tau_kv, float s_q, void* hip_stream) {
  if (B <= 0 || H <= 0 || L <= 0 || D <= 0 || block_q <= 0 || block_k <= 0)
    return sa_fail(SPARSE_ATTN_ERR_INVALID, "symbols: sizes must be positive (B=%d H=%d L=%d D=%d block_q=%d block_k=%d)", B, H,
                   L, D, block_q, block_k);
  if ((D != 64 && D != 128) || (block_q != 64 && block_q != 128) || (block_k != 64 && block_k != 128))
    return sa_fail(SPARSE_ATTN_ERR_UNSUPPORTED, "symbols: D, block_q and block_k must be 64 or 128 (got %d, %d, %d)", D,
                   block_q, block_k);
  if (granularity < 1 || granularity > 64)
    return sa_fail(SPARSE_ATTN_ERR_INVALID, "symbols: granularity=%d must be between 1 and 64", granularity);
  if (text_tokens <= 0 || text_tokens >= L)
    return sa_fail(SPARSE_ATTN_ERR_INVALID, "symbols: text_tokens=%d must leave text and vision tokens (L=%d)", text_tokens, L);
  // pooled blocks of n * b tokens; a short last block counts as a block, and a pooled block that holds any text
  // token counts as text (the ceiling of Section 3.3)
  const int pool_q = granularity * block_q, pool_k = granularity * block_k;
  const int Tq = (L + pool_q - 1) / pool_q, Tk = (L + pool_k - 1) / pool_k;
  const int n_tq = (text_tokens + pool_q - 1) / pool_q, n_tk = (text_tokens + pool_k - 1) / pool_k;
  if (n_tq >= Tq || n_tk >= Tk)
    return sa_fail(SPARSE_ATTN_ERR_INVALID, "symbols: no vision block is left (%d of %d query blocks and %d of %d key blocks are text)",
                   n_tq, Tq, n_tk, Tk);
  if (Tq > kMaxBlocks || Tk > kMaxBlocks)
    return sa_fail(SPARSE_ATTN_ERR_UNSUPPORTED, "symbols: %d x %d pooled blocks exceed %d", Tq, Tk, kMaxBlocks);
  if (!(tau_c >= 0.f && tau_c <= 1.f) || !(tau_kv >= 0.f && tau_kv <= 1.f) || !(s_q >= 0.f && s_q <= 1.f))
    return sa_fail(SPARSE_ATTN_ERR_INVALID, "symbols: tau_c, tau_kv and s_q must lie in [0, 1] (got %g, %g, %g)",
                   (double)tau_c, (double)tau_kv, (double)s_q);
  const long long BH = (long long)B * H;
  const long long n_q_blocks = BH * Tq, n_k_blocks = BH * Tk;
  if (BH * (Tq > Tk ? Tq : Tk) > 0x3fffffffLL)
    return sa_fail(SPARSE_ATTN_ERR_UNSUPPORTED, "symbols: too many blocks (%lld)", BH * (Tq > Tk ? Tq : Tk));
  if (!Q || !K || !cache_flags || !kv_mask)
    return sa_fail(SPARSE_ATTN_ERR_INVALID, "symbols: Q, K, cache_flags and kv_mask must not be NULL");
  if (((uintptr_t)Q | (uintptr_t)K) & 15) return sa_fail(SPARSE_ATTN_ERR_INVALID, "symbols: Q and K must be 16-byte aligned");

  hipStream_t stream = (hipStream_t)hip_stream;
  const size_t pooled_b = align256((size_t)(n_q_blocks + n_k_blocks) * D * 4);
  const size_t rows_b = align256((size_t)BH * n_tq * Tk * 4);
  const size_t cols_b = align256((size_t)BH * Tq * n_tk * 4);
  void* ws = nullptr;
  if (int rc = sa_get_scratch(pooled_b + rows_b + cols_b, stream, &ws)) return rc;
  float* pooled = (float*)ws;
  float* text_rows = (float*)((char*)ws + pooled_b);
  float* text_cols = (float*)((char*)ws + pooled_b + rows_b);

  const int row_bytes = (Tk + 7) / 8;
  const float scale = (float)(1.0 / sqrt((double)D));
  const int np = map_np(Tk);
  const int groups = (Tq + kMapRows - 1) / kMapRows;
  const int T_pad = (Tk + 3) & ~3;
  const size_t map_lds = (size_t)kMapRows * T_pad * 4;
  static std::once_flag attr_once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(attr_once, [] {
    constexpr int kMaxLds = kMapRows * kMaxBlocks * 4;
    attr_err = hipFuncSetAttribute((const void*)map_rows<128, 0>, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
    if (attr_err == hipSuccess)
      attr_err = hipFuncSetAttribute((const void*)map_rows<64, 0>, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
  });
  if (attr_err != hipSuccess)
    return sa_fail(SPARSE_ATTN_ERR_HIP, "hipFuncSetAttribute(map_rows) failed: %s", hipGetErrorString(attr_err));
  const unsigned pool_grid = (unsigned)(BH * (Tq > Tk ? Tq : Tk));
  auto pool = D == 128 ? pool_blocks<128> : pool_blocks<64>;
  hipLaunchKernelGGL(pool, dim3(pool_grid, 2), dim3(256), 0, stream, (const uint16_t*)Q, (const uint16_t*)K, pooled, pool_q,
                     pool_k, Tq, Tk, L, n_q_blocks);
  HIP_TRY(hipGetLastError());
  // rows are searched in registers, 16 lanes to a row; beyond 512 entries in LDS
  auto map = D == 128 ? map_for<128>(Tk) : map_for<64>(Tk);
  hipLaunchKernelGGL(map, dim3((unsigned)(BH * groups)), dim3(map_threads(np)), map_lds, stream, pooled, n_q_blocks, Tq, Tk, T_pad,
                     n_tq, n_tk, row_bytes, scale, tau_kv, kv_mask, text_rows, text_cols);
  HIP_TRY(hipGetLastError());
  // (entries per lane, 64 lanes to a row: 5 for the 258 blocks of 33024 tokens; more are searched in LDS)
  auto select = Tq <= 64 ? select_blocks<1> : Tq <= 128 ? select_blocks<2> : Tq <= 320 ? select_blocks<5> : select_blocks<0>;
  hipLaunchKernelGGL(select, dim3((unsigned)BH), dim3(256), 0, stream, text_rows, text_cols, Tq, Tk, n_tq, n_tk, pool_q, pool_k,
                     L, tau_c, s_q, cache_flags);
  HIP_TRY(hipGetLastError());
  return 0;
}

int sparse_symbols_update_stream(const void* Q, const void* K, uint8_t* cache_flags, uint8_t* kv_mask, int B, int H,
                                 int L, int D, int block, int text_tokens, float tau_c, float tau_kv, float s_q,
                                 void* hip_stream) {
  return sparse_symbols_update_granular(Q, K, cache_flags, kv_mask, B, H, L, D, block, block, 1, text_tokens, tau_c, tau_kv,
                                        s_q, hip_stream);
}

int sparse_symbols_update(const void* Q, const void* K, uint8_t* cache_flags, uint8_t* kv_mask, int B, int H, int L,
                          int D, int block, int text_tokens, float tau_c, float tau_kv, float s_q) {
  return sparse_symbols_update_stream(Q, K, cache_flags, kv_mask, B, H, L, D, block, text_tokens, tau_c, tau_kv, s_q,
                                      nullptr);
}

}  // extern "C"
