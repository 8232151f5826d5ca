// Sparse query projection (GEMM-Q of the paper, Section 3.5, Observation 2 / Equation 2) for gfx950.
//
// Q[b,h,i-th block,:] = X[b, i-th block, :] . W_h^T (+ bias_h) for every (b,h,i) whose cache flag is clear; a flagged
// block is left alone (its attention output is reused from the cache, so its queries are never read).  Without flags
// the product is tiled like a dense one (256 x 256: two heads at a time); with flags a tile is one head and two (or
// four) of its computed query blocks, found by ballots over the head's flags.  The product is computed transposed,
// C^T[d][token] = sum_k W[d][k] X[token][k], with v_mfma_f32_32x32x16_bf16: both operands are "k contiguous" rows (A =
// weight rows, B = token rows), so both come out of LDS with plain 16-byte reads, and a lane ends up holding 4
// consecutive d of one token.  The result leaves through LDS as whole rows of the [B,H,L,D] layout that the attention
// kernel reads.
//
// What bounds it (33024 tokens, C = 3072, 24 heads of 128, inputs that are not in the caches).  Dense: power; the
// matrix pipe is busy 67 % of the time at 1.66 GHz: 632 -> 508 us (1227 TFLOP/s), with RMSNorm and RoPE 737 -> 540 us; the
// 128 x 128 tiles it replaces streamed 64 KB from L2 per 1024 MFMA cycles of a CU, these 32.  80 % of the blocks cached:
// 166 us, matrix pipe busy 40 %, 0.95 GB fetched past L2 (a token block's rows are wanted by heads whose weights live on
// different XCDs) and 624 tiles on 256 CUs, 2.4 rounds; which of the two holds it back has not been separated.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "sparse_attn.h"
#include "sparse_attn_internal.h"

namespace {

using sa_gemm::f32x16;
using sa_gemm::kCus;
using sa_gemm::kRowB;
using sa_gemm::kStepK;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;

#define LDS_PTR(T) T __attribute__((address_space(3)))*
#define GLOBAL_PTR(T) T __attribute__((address_space(1)))*

struct GemmQParams {
  const char* X;       // bf16 [B, L, C]
  const char* W;       // bf16 [H*D, C]
  const uint16_t* bias;  // bf16 [H*D] or nullptr
  const uint8_t* flags;  // [B, H, Tq] or nullptr
  char* Q;             // bf16 [B, H, L, D]
  int H, L, C, Tq;
  int tok_begin, tok_end;   // tokens of every sequence that this launch works on (whole sequences where flags are given)
  // fused epilogue (NORM_ROPE instantiations only)
  const uint16_t* norm_w;   // bf16 [D] or nullptr (= ones)
  const float* rope_cos;    // fp32 [L, D/2] or nullptr (= no rotation)
  const float* rope_sin;
  float eps;
};

// TM tokens x TN channels per workgroup, WM x WN waves, WB / XB LDS buffers.  BQ > 0: the tokens are TM / BQ query
// blocks of one head (TN = D) whose flags are clear, wherever in the sequence they lie; BQ = 0: TM consecutive tokens.
template <int TM, int TN, int WM, int WN, int WB, int XB, int D, int BQ, bool NORM_ROPE>
__global__ void __launch_bounds__(WM * WN * 64, 2) gemm_q_kernel(const GemmQParams p) {
  using Pipe = sa_gemm::Pipe<TN, TM, WN, WM, WB, XB>;
  constexpr int NWAVES = WM * WN;
  constexpr int NT = NWAVES * 64;
  constexpr int A = Pipe::kA, C = Pipe::kC;
  constexpr int CW = TN / WN, TW = TM / WM;       // channels / tokens of a wave's corner
  constexpr int HPW = CW >= D ? CW / D : 1;       // heads of which a wave holds all channels (or one in part)
  constexpr int NB = CW >= D ? D / 32 : CW / 32;  // 32-channel blocks of a head in a wave
  constexpr int BR = BQ > 0 ? BQ : TM;            // consecutive tokens
  constexpr int NG = TM / BR;                     // runs of them
  static_assert(CW >= D || (CW * 2 == D && WN == 2), "a head lies in one wave or in two");
  static_assert(BQ == 0 || (TN == D && TM % BR == 0 && BR % TW == 0), "a gathered tile is whole blocks of one head");
  // LDS after the reduction loop: cos and sin rows of the tile, later the waves' output corners; behind them the bias
  // and gain as floats and the row sums of heads that lie in two waves
  constexpr int TABB = TM * (D / 2) * 4;          // bytes of one table
  constexpr int kVec = 2 * TABB > TM * TN * 2 ? 2 * TABB : TM * TN * 2;
  constexpr int kGain = kVec + TN * 4;
  constexpr int kPart = kGain + D * 4;

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const unsigned lds_base = (unsigned)(uintptr_t)(LDS_PTR(char))smem;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WM, wn = wave / WM;
  const int l32 = lane & 31, half = lane >> 5;

  // tile of this workgroup: column tile ct, batch b, and the token runs: first token, tokens that exist
  int ct, b;
  int tok0[NG], rows[NG];
  const int n_col = (p.H * D + TN - 1) / TN;
  if constexpr (BQ > 0) {
    // head fastest, so every XCD keeps the weights of a fixed set of heads in its L2; the tiles past a head's last
    // computed block come last in the grid
    const int n_tok = (p.Tq + NG - 1) / NG;
    ct = blockIdx.x % n_col;
    const int j = (blockIdx.x / n_col) % n_tok;
    b = blockIdx.x / (n_col * n_tok);
    // the computed blocks number NG * j .. NG * j + NG - 1 of this head: ballots over the flags, 64 blocks per wave
    const uint8_t* fr = p.flags + ((size_t)b * p.H + ct) * p.Tq;
    unsigned long long* const masks = (unsigned long long*)smem;
    int seen = 0, blk[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) blk[g] = -1;
    for (int c0 = 0; c0 < p.Tq && blk[NG - 1] < 0; c0 += NT) {
      const unsigned long long live = __builtin_amdgcn_ballot_w64(c0 + tid < p.Tq && fr[min(c0 + tid, p.Tq - 1)] == 0);
      if (lane == 0) masks[wave] = live;
      __syncthreads();
      for (int w = 0; w < NWAVES; ++w) {
        const unsigned long long mv = masks[w];
        // (readfirstlane returns int: through unsigned, or bit 31 would be spread over the upper word)
        const unsigned m_lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)mv);
        const unsigned m_hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(mv >> 32));
        const unsigned long long m = (unsigned long long)m_hi << 32 | m_lo;
        const int count = __popcll(m);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const int rank = NG * j + g - seen;     // among the set bits of this word
          if (rank >= 0 && rank < count) {
            const bool here = ((m >> lane) & 1ull) && __popcll(m & ((1ull << lane) - 1ull)) == rank;
            blk[g] = c0 + 64 * w + __builtin_ctzll(__builtin_amdgcn_ballot_w64(here));
          }
        }
        seen += count;
      }
      __syncthreads();                            // the masks are rewritten, or a stage lands on them
    }
    if (blk[0] < 0) return;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      tok0[g] = (blk[g] < 0 ? blk[0] : blk[g]) * BR;   // a missing block re-reads the first one
      rows[g] = blk[g] < 0 ? 0 : min(BR, p.L - tok0[g]);
    }
  } else {
    const int n_tok = (p.tok_end - p.tok_begin + TM - 1) / TM;
    int i;
    if constexpr (TN > 128) {
      // The 8 XCDs (workgroup n runs on XCD n mod 8) take a contiguous part each of the tiles in the order: batch,
      // group of 4 column tiles, token tile, column tile.  The 32 tiles an XCD works on at a time are then 4 column
      // tiles x 8 token tiles: the stage loads of 12 operand tiles serve 32 workgroups.
      const int tiles = (int)gridDim.x, x = blockIdx.x % 8, at = blockIdx.x / 8;
      int n = x * (tiles / 8) + min(x, tiles % 8) + at;
      b = n / (n_col * n_tok);
      n -= b * (n_col * n_tok);
      const int g = n / (4 * n_tok), width = min(4, n_col - 4 * g);
      n -= g * 4 * n_tok;
      i = n / width;
      ct = 4 * g + n % width;
    } else {
      // column tile fastest: every XCD keeps the weights of a fixed set of column tiles in its L2
      ct = blockIdx.x % n_col;
      i = (blockIdx.x / n_col) % n_tok;
      b = blockIdx.x / (n_col * n_tok);
    }
    tok0[0] = p.tok_begin + i * TM;
    rows[0] = min(TM, p.tok_end - tok0[0]);       // the last token tile may be short
  }
  // first token and rows of the run that tile row r lies in
  auto pick = [](const int (&v)[NG], int g) {
    // (all values first: a choice between elements would put the array into scratch memory)
    const int v0 = v[0], v1 = v[NG > 1 ? 1 : 0], v2 = v[NG > 2 ? 2 : 0], v3 = v[NG > 2 ? 3 : 0];
    const int lo = NG > 1 && (g & 1) ? v1 : v0, hi = NG > 2 && (g & 1) ? v3 : v2;
    return NG > 2 && (g & 2) ? hi : lo;
  };
  static_assert(NG == 1 || NG == 2 || NG == 4, "pick() knows these");
  auto run_tok0 = [&](int r) { return pick(tok0, r / BR); };
  auto run_rows = [&](int r) { return pick(rows, r / BR); };

  const size_t row_pitch = (size_t)p.C * 2;
  const int n0 = ct * TN;                         // first output channel of the tile
  const int cols_valid = min(TN, p.H * D - n0);   // the last column tile may be short
  const char* gW = p.W + (size_t)n0 * row_pitch;
  Pipe st;
  st.init(lds_base, wave, lane, wn, wm, row_pitch, cols_valid);
#pragma unroll
  for (int u = 0; u < Pipe::kXLoad; ++u) {
    // a load covers 8 rows of one run; rows that do not exist re-read the last one that does and are never stored
    const int r0 = (wave + u * NWAVES) * 8, r = r0 + lane / 8;
    st.set_x_rows(u, sa_uniform_ptr(p.X + ((size_t)b * p.L + run_tok0(r0)) * row_pitch),
                  min(r % BR, max(run_rows(r0), 1) - 1), row_pitch, lane);
  }

  f32x16 acc[A][C];   // [channel block][token block] of this wave's corner
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[a][c][e] = 0.f;

  // The tile's cos / sin rows, 16-byte pieces.  They are requested behind the last stage and land under its MFMAs (256 x
  // 256 tiles have no registers for that: there they are requested behind the loop).
  constexpr int CHT = D / 8;                      // 16-byte chunks of a table row
  constexpr int PER = TABB / 16 / NT;             // pieces of a table per thread
  static_assert(TABB % (16 * NT) == 0, "table pieces must split evenly over the threads");
  constexpr bool kEarly = A * C < 8;
  f32x4 vc[kEarly ? PER : 1], vs[kEarly ? PER : 1];
  // piece u of this thread: a wave's 64 lie in one run, whose first token is a uniform 64-bit offset (a table may be
  // larger than 4 GiB); the rest fits in 32 bits.  The tables need 8-byte alignment only.
  typedef f32x4 __attribute__((aligned(8))) f32x4_a8;
  auto table_piece = [&](const float* table, int u) -> f32x4 {
    const int r0 = (u * NT + wave * 64) / CHT, row = (u * NT + tid) / CHT;
    const char* base = sa_uniform_ptr((const char*)table + (size_t)run_tok0(r0) * (CHT * 16));
    const unsigned off = (unsigned)(min(row % BR, max(run_rows(r0), 1) - 1) * CHT + tid % CHT) * 16;
    return *(GLOBAL_PTR(const f32x4_a8))(base + off);   // (the address space got lost in sa_uniform_ptr)
  };
  auto prefetch_tables = [&]() -> int {
    if constexpr (NORM_ROPE && kEarly) {
      if (p.rope_cos) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          vc[u] = table_piece(p.rope_cos, u);
          vs[u] = table_piece(p.rope_sin, u);
        }
        return 2 * PER;
      }
    }
    return 0;
  };

  // Bias and gain of the tile, one value per thread, in flight during the reduction (256 x 256 tiles have no registers
  // for that either).  Loaded without a branch -- from the weights where there is none -- and converted behind the
  // loop, so that nothing waits for them here.
  const uint16_t* const bias_p = p.bias ? p.bias : (const uint16_t*)p.W;
  const uint16_t* const gain_p = p.norm_w ? p.norm_w : (const uint16_t*)p.W;
  auto load_bias = [&]() -> unsigned { return bias_p[min(n0 + min(tid, TN - 1), p.H * D - 1)]; };
  auto load_gain = [&]() -> unsigned { return gain_p[min(tid, D - 1)]; };
  unsigned bias_bits = 0, gain_bits = 0;
  if constexpr (kEarly) {
    bias_bits = load_bias();
    if constexpr (NORM_ROPE) gain_bits = load_gain();
  }

  size_t k_off = 0;
  st.run(
      smem, acc, p.C / kStepK,
      [&]() {
        const char* at = gW;
        gW += kRowB;
        return at;
      },
      [&]() {
        const size_t at = k_off;
        k_off += kRowB;
        return at;
      },
      prefetch_tables);
  __syncthreads();                                // every wave is done reading the operand stages

  // ---- epilogue: lane holds token 32 * c + l32 and, per accumulator quad q4, channels 32 * a + 8 * q4 + 4 * half
  // + 0..3 of this wave's corner
  float* const bias_f = (float*)(smem + kVec);
  float* const gain_f = (float*)(smem + kGain);
  static_assert(TN <= NT && D <= NT, "one bias and one gain value per thread");
  if constexpr (!kEarly) {
    bias_bits = load_bias();
    if constexpr (NORM_ROPE) gain_bits = load_gain();
  }
  if (tid < TN) bias_f[tid] = p.bias ? __builtin_bit_cast(float, bias_bits << 16) : 0.f;
  auto tab_swizzle = [](int row) { return CHT == 16 ? (row & 15) : ((row >> 1) & 7); };
  if constexpr (NORM_ROPE) {
    if (tid < D) gain_f[tid] = p.norm_w ? __builtin_bit_cast(float, gain_bits << 16) : 1.f;
    // The tile's cos / sin rows come through LDS: read straight from memory in the accumulator layout, every lane would
    // fetch 8 bytes from its own row.  16-byte chunks are permuted by the token so that the 32 tokens of a read spread
    // over the banks.
    if (p.rope_cos) {
      auto put = [&](int u, f32x4 c, f32x4 n) {
        const int e = u * NT + tid, row = e / CHT;
        const int o = row * CHT * 16 + ((e % CHT) ^ tab_swizzle(row)) * 16;
        *(f32x4*)(smem + o) = c;
        *(f32x4*)(smem + TABB + o) = n;
      };
      if constexpr (kEarly) {
#pragma unroll
        for (int u = 0; u < PER; ++u) put(u, vc[u], vs[u]);
      } else {
        f32x4 c[PER], n[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          c[u] = table_piece(p.rope_cos, u);
          n[u] = table_piece(p.rope_sin, u);
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) put(u, c[u], n[u]);
      }
    }
  }
  __syncthreads();
  // (without a bias zeros are added: a branch here makes the compiler keep the accumulators twice)
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const float4 bv = *(const float4*)(bias_f + wn * CW + 32 * a + 8 * q4 + 4 * half);
#pragma unroll
      for (int c = 0; c < C; ++c) {
        acc[a][c][4 * q4 + 0] += bv.x;
        acc[a][c][4 * q4 + 1] += bv.y;
        acc[a][c][4 * q4 + 2] += bv.z;
        acc[a][c][4 * q4 + 3] += bv.w;
      }
    }
  if constexpr (NORM_ROPE) {
    // Equation 2: token-wise RMS normalisation over the head's D channels, then the rotation.  A token's sum of
    // squares is spread over this lane's values, the lane 32 further on, and the other wave of a head in two waves.
    float inv_rms[C][HPW];
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int hh = 0; hh < HPW; ++hh) {
        float v = 0.f;
#pragma unroll
        for (int a = hh * NB; a < (hh + 1) * NB; ++a)
#pragma unroll
          for (int e = 0; e < 16; ++e) v = fmaf(acc[a][c][e], acc[a][c][e], v);
        inv_rms[c][hh] = v + __shfl_xor(v, 32);
      }
    if constexpr (CW < D) {
      float* part = (float*)(smem + kPart);       // [WN][TM]
#pragma unroll
      for (int c = 0; c < C; ++c)
        if (half == 0) part[wn * TM + wm * TW + 32 * c + l32] = inv_rms[c][0];
      __syncthreads();
#pragma unroll
      for (int c = 0; c < C; ++c) inv_rms[c][0] = part[wm * TW + 32 * c + l32] + part[TM + wm * TW + 32 * c + l32];
    }
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int hh = 0; hh < HPW; ++hh) inv_rms[c][hh] = 1.0f / sqrtf(inv_rms[c][hh] * (1.0f / D) + p.eps);
#pragma unroll
    for (int a = 0; a < A; ++a)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int d0 = (wn * CW + 32 * a + 8 * q4 + 4 * half) % D;     // channel inside the head
        const float4 gain = *(const float4*)(gain_f + d0);
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const float inv = inv_rms[c][a / NB % HPW];
          float y0 = acc[a][c][4 * q4 + 0] * inv * gain.x, y1 = acc[a][c][4 * q4 + 1] * inv * gain.y;
          float y2 = acc[a][c][4 * q4 + 2] * inv * gain.z, y3 = acc[a][c][4 * q4 + 3] * inv * gain.w;
          if (p.rope_cos) {
            // channels d0..d0+3 are the pairs d0/2 and d0/2 + 1 of this token
            const int row = wm * TW + 32 * c + l32;
            const char* at = smem + row * CHT * 16 + ((d0 / 8) ^ tab_swizzle(row)) * 16 + 8 * half;
            const float2 cs = *(const float2*)at, sn = *(const float2*)(at + TABB);
            const float r0 = y0 * cs.x - y1 * sn.x, r1 = y0 * sn.x + y1 * cs.x;
            const float r2 = y2 * cs.y - y3 * sn.y, r3 = y2 * sn.y + y3 * cs.y;
            y0 = r0; y1 = r1; y2 = r2; y3 = r3;
          }
          acc[a][c][4 * q4 + 0] = y0;
          acc[a][c][4 * q4 + 1] = y1;
          acc[a][c][4 * q4 + 2] = y2;
          acc[a][c][4 * q4 + 3] = y3;
        }
      }
    __syncthreads();                              // every wave is done with the tables
  }
  // Output side.  A lane holds 4 channels of one token: written from here a store would be 8 bytes per lane, a row
  // apart.  Every wave sends its corner through a piece of LDS of its own (rows of CW bf16, 16-byte chunks permuted by
  // the token so that the 32 tokens of a write hit different banks) and stores whole rows, 16 bytes per lane, with
  // non-temporal stores: the projection writes its result once and must not push the weights and token rows out of
  // L2 with it.
  constexpr int CHO = CW / 8;                     // 16-byte chunks per row of the corner
  auto out_swizzle = [](int row) { return CHO == 16 ? (row & 15) : ((row >> 1) & 7); };
  char* const corner = smem + wave * TW * CW * 2;
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const int row = 32 * c + l32;
        bf16x2 lo, hi;
        lo[0] = (__bf16)acc[a][c][4 * q4 + 0];
        lo[1] = (__bf16)acc[a][c][4 * q4 + 1];
        hi[0] = (__bf16)acc[a][c][4 * q4 + 2];
        hi[1] = (__bf16)acc[a][c][4 * q4 + 3];
        u32x2 pk;
        pk[0] = __builtin_bit_cast(unsigned, lo);
        pk[1] = __builtin_bit_cast(unsigned, hi);
        *(u32x2*)(corner + row * CW * 2 + (((4 * a + q4) ^ out_swizzle(row)) * 16) + 8 * half) = pk;
      }
  // (only this wave touches its corner: LDS accesses of a wave execute in order)
#pragma unroll
  for (int it = 0; it < TW * CHO / 64; ++it) {
    const int row = it * (64 / CHO) + lane / CHO, ch = lane % CHO;
    const u32x4 v = *(const u32x4*)(corner + row * CW * 2 + ((ch ^ out_swizzle(row)) * 16));
    const int r = wm * TW + row, n = wn * CW + ch * 8;                 // inside the tile
    const int h = (n0 + n) / D, d = (n0 + n) % D;
    char* const out = p.Q + ((((size_t)b * p.H + h) * p.L + run_tok0(wm * TW) + r % BR) * D + d) * 2;
    if (r % BR < run_rows(wm * TW) && n < cols_valid) __builtin_nontemporal_store(v, (u32x4*)out);
  }
}

template <int TM, int TN, int WM, int WN, int WB, int XB, int D, int BQ, bool NORM_ROPE>
int launch_tiles(const GemmQParams& p, int B, hipStream_t stream) {
  constexpr size_t stage_lds = sa_gemm::Pipe<TN, TM, WN, WM, WB, XB>::kLdsBytes;
  constexpr size_t out_lds = TM * D * 4 > TM * TN * 2 ? (size_t)TM * D * 4 : (size_t)TM * TN * 2;
  constexpr size_t epi_lds = out_lds + (TN + D + WN * TM) * 4;
  constexpr size_t lds = stage_lds > epi_lds ? stage_lds : epi_lds;
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  constexpr int threads = WM * WN * 64;
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [] {
    attr_err = hipFuncSetAttribute((const void*)gemm_q_kernel<TM, TN, WM, WN, WB, XB, D, BQ, NORM_ROPE>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  });
  if (attr_err != hipSuccess)
    return sa_fail(SPARSE_ATTN_ERR_HIP, "hipFuncSetAttribute failed: %s", hipGetErrorString(attr_err));
  const int n_tok = BQ > 0 ? (p.Tq + TM / (BQ > 0 ? BQ : 1) - 1) / (TM / (BQ > 0 ? BQ : 1)) : (p.tok_end - p.tok_begin + TM - 1) / TM;
  const int tiles = B * n_tok * ((p.H * D + TN - 1) / TN);
  hipLaunchKernelGGL((gemm_q_kernel<TM, TN, WM, WN, WB, XB, D, BQ, NORM_ROPE>), dim3(tiles), dim3(threads), lds, stream, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return sa_fail(SPARSE_ATTN_ERR_HIP, "gemm_q launch failed: %s", hipGetErrorString(e));
  return 0;
}

// Which tile.  One workgroup of the 256-token kernels fills a CU, two of the 128 x 128 one do; the figures are the
// plain projection at C = 3072, us.
//   no flags   up to 256 tiles of 128 x 128 (one per CU): those (24 heads x 1024 tokens: 28 against 32 and 55 for the
//              two larger tiles); up to 512: 256 x 128 (2048 tokens: 41 against 44 and 57); beyond: 256 x 256, which
//              asks L2 for half as many bytes per product (4608 tokens: 72 against 82 and 84; 33024: 528 against 587
//              and 605).  A last round of 256 x 256 tiles that would be less than half full is done with the smaller
//              tiles instead (33024 tokens are 6.05 rounds: 508).
//   flags      two (block_q 64: four) computed blocks of one head share their weight rows: 33024 tokens, 80 % cached:
//              161 against 187 with a tile per block, 4608 tokens, 56 %: 43 against 63.  Few tiles in all: one per block.
template <int D, bool NR>
int launch(GemmQParams p, int B, int block_q, hipStream_t stream) {
  const int heads_per_128 = 128 / D;
  if (!p.flags) {
    const int tok = p.tok_end - p.tok_begin;
    const long long units = (long long)B * ((tok + 127) / 128) * ((p.H + heads_per_128 - 1) / heads_per_128);
    if (units <= kCus) return launch_tiles<128, 128, 2, 2, 2, 3, D, 0, NR>(p, B, stream);
    if (units <= 2 * kCus) return launch_tiles<256, 128, 4, 2, 3, 3, D, 0, NR>(p, B, stream);
    const int n_col = (p.H * D + 255) / 256, n_tok = (tok + 255) / 256;
    const long long tiles = (long long)B * n_tok * n_col, full = tiles / kCus * kCus;
    const int keep = (int)(full / ((long long)B * n_col));         // token tiles per sequence that fill whole rounds
    if (tiles > full && tiles - full <= kCus / 2 && keep > 0) {
      GemmQParams rest = p;
      p.tok_end = rest.tok_begin = p.tok_begin + keep * 256;
      if (int rc = launch_tiles<256, 256, 4, 2, 2, 3, D, 0, NR>(p, B, stream)) return rc;
      return launch<D, NR>(rest, B, block_q, stream);
    }
    return launch_tiles<256, 256, 4, 2, 2, 3, D, 0, NR>(p, B, stream);
  }
  const long long blocks = (long long)B * p.H * p.Tq;
  if constexpr (D == 128) {
    if (block_q == 128) {
      if (blocks <= kCus) return launch_tiles<128, 128, 2, 2, 2, 3, 128, 128, NR>(p, B, stream);
      return launch_tiles<256, 128, 4, 2, 3, 3, 128, 128, NR>(p, B, stream);
    }
    if (blocks <= 2 * kCus) return launch_tiles<128, 128, 2, 2, 2, 3, 128, 64, NR>(p, B, stream);
    return launch_tiles<256, 128, 4, 2, 3, 3, 128, 64, NR>(p, B, stream);
  } else {
    if (block_q == 128) {
      if (blocks <= 2 * kCus) return launch_tiles<128, 64, 2, 1, 2, 3, 64, 128, NR>(p, B, stream);
      return launch_tiles<256, 64, 4, 1, 2, 2, 64, 128, NR>(p, B, stream);
    }
    if (blocks <= 2 * kCus) return launch_tiles<64, 64, 1, 1, 2, 3, 64, 64, NR>(p, B, stream);
    if (blocks <= 4 * kCus) return launch_tiles<128, 64, 2, 1, 2, 3, 64, 64, NR>(p, B, stream);
    return launch_tiles<256, 64, 4, 1, 2, 2, 64, 64, NR>(p, B, stream);
  }
}

bool ranges_overlap(const void* a, size_t na, const void* b, size_t nb) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + nb && y < x + na;
}

int gemm_q_run(const void* X, const void* W, const void* bias, const uint8_t* cache_flags, void* Q, int B, int L, int C,
               int H, int D, int block_q, hipStream_t stream, bool norm_rope, const void* norm_weight, float eps,
               const float* rope_cos, const float* rope_sin) {
  if (B <= 0 || L <= 0 || C <= 0 || H <= 0 || D <= 0 || block_q <= 0)
    return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_q: sizes must be positive (B=%d L=%d C=%d H=%d D=%d block_q=%d)", B,
                   L, C, H, D, block_q);
  if ((D != 64 && D != 128) || (block_q != 64 && block_q != 128))
    return sa_fail(SPARSE_ATTN_ERR_UNSUPPORTED, "gemm_q: D and block_q must be 64 or 128 (got %d, %d)", D, block_q);
  if (C % kStepK) return sa_fail(SPARSE_ATTN_ERR_UNSUPPORTED, "gemm_q: C=%d must be a multiple of %d", C, kStepK);
  if ((long long)128 * C * 2 >= (1LL << 31)) return sa_fail(SPARSE_ATTN_ERR_UNSUPPORTED, "gemm_q: C=%d too large", C);
  const int tq = (L + block_q - 1) / block_q;      // a short last block counts as a block
  const long long tiles = (long long)B * H * tq;
  if (tiles > 0x3fffffffLL) return sa_fail(SPARSE_ATTN_ERR_UNSUPPORTED, "gemm_q: too many tiles (%lld)", tiles);
  if (!X || !W || !Q) return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_q: X, W and Q must not be NULL");
  if (((uintptr_t)X | (uintptr_t)W | (uintptr_t)Q) & 15)
    return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_q: X, W and Q must be 16-byte aligned");
  const size_t xb = (size_t)B * L * C * 2, wb = (size_t)H * D * C * 2, qb = (size_t)B * H * L * D * 2;
  if (ranges_overlap(Q, qb, X, xb) || ranges_overlap(Q, qb, W, wb))
    return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_q: Q must not overlap X or W");
  if (norm_rope) {
    if (!(eps >= 0.f) || eps - eps != 0.f) return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_q: eps must be finite and >= 0");
    if ((rope_cos == nullptr) != (rope_sin == nullptr))
      return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_q: rope_cos and rope_sin must be given together");
    if (((uintptr_t)rope_cos | (uintptr_t)rope_sin) & 7)
      return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_q: rope_cos and rope_sin must be 8-byte aligned");
    if ((uintptr_t)norm_weight & 1) return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_q: norm_weight must be 2-byte aligned");
  }

  GemmQParams p;
  p.X = (const char*)X;
  p.W = (const char*)W;
  p.bias = (const uint16_t*)bias;
  p.flags = cache_flags;
  p.Q = (char*)Q;
  p.H = H;
  p.L = L;
  p.C = C;
  p.Tq = tq;
  p.tok_begin = 0;
  p.tok_end = L;
  p.norm_w = (const uint16_t*)norm_weight;
  p.rope_cos = rope_cos;
  p.rope_sin = rope_sin;
  p.eps = eps;
  if (norm_rope) return D == 128 ? launch<128, true>(p, B, block_q, stream) : launch<64, true>(p, B, block_q, stream);
  return D == 128 ? launch<128, false>(p, B, block_q, stream) : launch<64, false>(p, B, block_q, stream);
}

}  // namespace

extern "C" {

int sparse_gemm_q_stream(const void* X, const void* W, const void* bias, const uint8_t* cache_flags, void* Q, int B,
                         int L, int C, int H, int D, int block_q, void* hip_stream) {
  return gemm_q_run(X, W, bias, cache_flags, Q, B, L, C, H, D, block_q, (hipStream_t)hip_stream, false, nullptr, 0.f,
                    nullptr, nullptr);
}

int sparse_gemm_q(const void* X, const void* W, const void* bias, const uint8_t* cache_flags, void* Q, int B, int L,
                  int C, int H, int D, int block_q) {
  return sparse_gemm_q_stream(X, W, bias, cache_flags, Q, B, L, C, H, D, block_q, nullptr);
}

int sparse_gemm_q_norm_rope(const void* X, const void* W, const void* bias, const void* norm_weight, float eps,
                            const float* rope_cos, const float* rope_sin, const uint8_t* cache_flags, void* Q, int B,
                            int L, int C, int H, int D, int block_q, void* hip_stream) {
  return gemm_q_run(X, W, bias, cache_flags, Q, B, L, C, H, D, block_q, (hipStream_t)hip_stream, true, norm_weight, eps,
                    rope_cos, rope_sin);
}

}  // extern "C"
