// Sparse output projection (GEMM-O of the paper, Section 3.5, Observation 3 / Equations 3-4) for gfx950.
//
// Out[b, token, n] = addend[b, token, n] + bias[n] + sum over SELECTED heads h of O[b,h,token,:] . W[n, h*D:(h+1)*D]
// where, for the token block i the token lies in, head h is selected when its cache flag equals
// `select`.  The paper's two stages are two calls: stage 1 at an Update step (select = flag set,
// no addend) produces the cached bias B_c, the part of the projection that comes from heads whose
// attention output is reused; stage 2 at every step (select = flag clear, addend = B_c) adds the
// heads that were really computed.  The skipping is along the REDUCTION axis: the K loop of a tile
// walks a bitmap of that token block's selected heads (built with one wave ballot, walked with
// scalar find-first-set) and never loads the O or W columns of the others.
//
// The addend may also be given as the stored terms of the cached bias and their weights: the kernel then forms
// OP_reuse(B_c) = sum_d coef[d] * terms[d] itself while it fetches them (fp32, term order, rounded to bf16 exactly
// as the stand-alone element-wise kernel rounds it), so a Dispatch step needs no separate pass that writes the
// forecast bias and reads it back.  A token block none of whose heads is selected only streams: addend + bias.
//
// One workgroup per (token tile, column tile); transposed MFMA product and staging as in the query projection (A =
// weight rows, B = token rows, both k-contiguous in LDS).
//
// What bounds it (33024 tokens, 24 heads of 128, 3072 channels).  90 % cached heads, two terms: 650 MB, 126 us at the rate
// of a large copy; 151 us: a tile is a chain of flags, first stage, five stages on average, addend and store, each a
// round trip to memory, with two tiles per CU to hide them.  No flags: power, as the query projection.
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

constexpr int kBN = 128;                   // C_out is a multiple of this
constexpr int kMaxTerms = 4;               // stored feature + up to three derivatives

struct GemmOParams {
  const char* O;         // bf16 [B, H, L, D]
  const char* W;         // bf16 [C_out, H*D]
  const uint16_t* bias;  // bf16 [C_out] or nullptr
  const uint8_t* flags;  // [B, H, Tq] or nullptr
  const char* addend;    // bf16 [B, L, C_out] or nullptr; with n_terms > 0: the first term
  char* Out;             // bf16 [B, L, C_out]
  int H, L, C_out, select;
  int tok_begin, tok_end;  // tokens of every sequence that this launch works on (whole sequences where flags are given)
  // OP_reuse of the cached bias fused into the addend: addend = sum_d coef[d] * term[d], term[0] = `addend`
  const char* term[kMaxTerms - 1];
  float coef[kMaxTerms];
  int n_terms;           // 0: `addend` is taken as it is
};

__device__ __forceinline__ float bf16_bits_to_float(unsigned bits16) {
  return __builtin_bit_cast(float, bits16 << 16);
}

// TM tokens x TN output channels per workgroup, WM x WN waves, WB / XB LDS buffers.  FLAGGED: the tokens are one token
// block (TM = block_q) and the reduction visits the heads its flags select; otherwise TM consecutive tokens and all heads.
// TWO: there may be a second term of the addend to request early; without it (FLAGGED) the loop for few stages is used.
template <int TM, int TN, int WM, int WN, int WB, int XB, int D, bool FLAGGED, bool TWO>
__global__ void __launch_bounds__(WM * WN * 64, 2) gemm_o_kernel(const GemmOParams p) {
  using Pipe = sa_gemm::Pipe<TN, TM, WN, WM, WB, XB>;
  constexpr int NWAVES = WM * WN;
  constexpr int A = Pipe::kA, C = Pipe::kC;
  constexpr int CW = TN / WN, TW = TM / WM;       // channels / tokens of a wave's corner
  constexpr int PARTS = D / kStepK;               // stages per head

  // tile of this workgroup
  const int n_col = (p.C_out + TN - 1) / TN, n_tok = (p.tok_end - p.tok_begin + TM - 1) / TM;
  int col, i, b;
  if constexpr (!FLAGGED && TN > 128) {
    // as in the query projection: every XCD takes a contiguous part of the tiles in the order batch, group of 4 column
    // tiles, token tile, column tile
    const int tiles = (int)gridDim.x, x = blockIdx.x % 8, at = blockIdx.x / 8;
    int n = x * (tiles / 8) + min(x, tiles % 8) + at;
    b = n / (n_col * n_tok);
    n -= b * (n_col * n_tok);
    const int g = n / (4 * n_tok), width = min(4, n_col - 4 * g);
    n -= g * 4 * n_tok;
    i = n / width;
    col = 4 * g + n % width;
  } else {
    // column tile fastest: the 8 XCDs (workgroup n runs on XCD n mod 8) each keep the weight rows of a fixed set of
    // column tiles in their L2 while the token blocks stream past
    col = blockIdx.x % n_col;
    i = (blockIdx.x / n_col) % n_tok;
    b = blockIdx.x / (n_col * n_tok);
  }
  const int tok0 = p.tok_begin + i * TM;

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const unsigned lds_base = (unsigned)(uintptr_t)(LDS_PTR(char))smem;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WM, wn = wave / WM;
  const int l32 = lane & 31, half = lane >> 5;

  // reduction-axis symbol of this token block: one bit per head, set = visit
  unsigned long long heads;
  if constexpr (FLAGGED) {
    bool mine = false;
    if (lane < p.H) mine = (p.flags[((size_t)b * p.H + lane) * n_tok + i] != 0 ? 1 : 0) == p.select;
    heads = __builtin_amdgcn_ballot_w64(mine);
  } else {
    heads = p.select ? 0ull : (p.H == 64 ? ~0ull : (1ull << p.H) - 1ull);   // no flags: no head counts as cached
  }

  const size_t w_pitch = (size_t)p.H * D * 2;
  const int n0 = col * TN;                        // first output channel of the tile
  // the last token tile and the last column tile may be short: loads of missing rows re-read the last row that
  // exists, their results are never stored
  const int rows_valid = min(TM, p.tok_end - tok0), cols_valid = min(TN, p.C_out - n0);
  const char* gW = p.W + (size_t)n0 * w_pitch;
  Pipe st;
  st.init(lds_base, wave, lane, wn, wm, w_pitch, cols_valid);
  {
    const char* gO = sa_uniform_ptr(p.O + ((size_t)b * p.H * p.L + tok0) * (size_t)(D * 2));   // head 0; head h adds h*L*D*2
#pragma unroll
    for (int u = 0; u < Pipe::kXLoad; ++u)
      st.set_x_rows(u, gO, min(Pipe::load_row(wave, lane, u), rows_valid - 1), (size_t)(D * 2), lane);
  }

  f32x16 acc[A][C];   // [output-channel block][token block] of this wave's corner
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[a][c][e] = 0.f;

  // Output side: thread -> (row, group of 8 output channels), whole rows of the tile at a time (256 x 256 tiles: of the
  // wave's corner), for the addend's loads as for the result's stores; both are streamed once: non-temporal, so that they
  // do not push the weight rows out of the XCD's L2.
  constexpr bool kWhole = TM * TN * 4 <= 160 * 1024;   // the tile fits into LDS in fp32
  constexpr int kLanes = kWhole ? NWAVES * 64 : 64;
  constexpr int CHO = (kWhole ? TN : CW) / 8;     // 16-byte pieces per row
  constexpr int RPI = kLanes / CHO;               // rows per pass
  constexpr int OUT_ITERS = (kWhole ? TM : TW) / RPI;
  const int out_row = tid % kLanes / CHO, out_ch = tid % CHO;
  const int row0 = kWhole ? 0 : wm * TW, col0 = kWhole ? 0 : wn * CW;
  const size_t out0 = (((size_t)b * p.L + tok0 + row0) * p.C_out + n0 + col0) * 2;
  auto out_offset = [&](int it) -> size_t { return out0 + ((size_t)(it * RPI + out_row) * p.C_out + out_ch * 8) * 2; };
  auto there = [&](int it) -> bool { return row0 + it * RPI + out_row < rows_valid && col0 + out_ch * 8 < cols_valid; };

  // The first two terms of the addend are requested behind the last stage of the reduction and land under its MFMAs;
  // their OP_reuse is formed in the epilogue.  Loads return in order, so requested earlier they would hold up the
  // stages behind them (128 x 128 tiles, 33024 tokens, one term, 4 heads per block: 153 us; 165 when requested behind the
  // first stages).  The loop for few stages asks for its one term behind the first stage.  Returns the number of loads
  // where it is certain: in a tile at the edge a wave may skip some.  (256 x 256 tiles have no registers for that: there
  // the addend is requested behind the loop.)
  static_assert(!kWhole || OUT_ITERS == 8, "the loops count on 8 or 16 loads");
  u32x4 term0[OUT_ITERS], term1[kWhole && TWO ? OUT_ITERS : 1];
  const bool two = kWhole && TWO && p.n_terms > 1;
  auto fetch_addend = [&]() __attribute__((always_inline)) -> int {
    if (!p.addend) return 0;
    if (rows_valid == TM && cols_valid == TN) {
#pragma unroll
      for (int it = 0; it < OUT_ITERS; ++it) term0[it] = __builtin_nontemporal_load((const u32x4*)(p.addend + out_offset(it)));
      if (!two) return OUT_ITERS;
#pragma unroll
      for (int it = 0; it < OUT_ITERS; ++it) term1[kWhole && TWO ? it : 0] = __builtin_nontemporal_load((const u32x4*)(p.term[0] + out_offset(it)));
      return 2 * OUT_ITERS;
    }
#pragma unroll
    for (int it = 0; it < OUT_ITERS; ++it) {
      if (!there(it)) continue;
      term0[it] = __builtin_nontemporal_load((const u32x4*)(p.addend + out_offset(it)));
      if (two) term1[kWhole && TWO ? it : 0] = __builtin_nontemporal_load((const u32x4*)(p.term[0] + out_offset(it)));
    }
    return 0;
  };
  // the addend of one piece: as given, or OP_reuse(B_c): fp32 sum of the scaled terms in term order, one rounding to
  // bf16 (what the element-wise kernel computes)
  auto addend_of = [&](int it) __attribute__((always_inline)) -> u32x4 {
    u32x4 r = term0[it];
    if (p.n_terms > 0) {
      float v[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[2 * e] = p.coef[0] * bf16_bits_to_float(term0[it][e] & 0xffffu);
        v[2 * e + 1] = p.coef[0] * bf16_bits_to_float(term0[it][e] >> 16);
      }
      for (int d = 1; d < p.n_terms; ++d) {
        const u32x4 tb = kWhole && TWO && d == 1 ? term1[kWhole && TWO ? it : 0] : __builtin_nontemporal_load((const u32x4*)(p.term[d - 1] + out_offset(it)));
        const float cd = p.coef[d];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[2 * e] = fmaf(cd, bf16_bits_to_float(tb[e] & 0xffffu), v[2 * e]);
          v[2 * e + 1] = fmaf(cd, bf16_bits_to_float(tb[e] >> 16), v[2 * e + 1]);
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        bf16x2 pr;
        pr[0] = (__bf16)v[2 * e];
        pr[1] = (__bf16)v[2 * e + 1];
        r[e] = __builtin_bit_cast(unsigned, pr);
      }
    }
    return r;
  };

  // Bias, in flight during the reduction: loaded without a branch -- from the weights where there is none -- and converted
  // behind the loop, so that nothing waits for it here.  A thread's 8 channels in one load (at the 2-byte alignment of the
  // bias: eight loads of 2 bytes would be as many requests as a tile without a head has stores), or the channels of
  // the corner, one per lane.
  typedef u32x4 __attribute__((aligned(2))) u32x4_a2;
  const uint16_t* const bias_p = p.bias ? p.bias : (const uint16_t*)p.W;
  const u32x4 bias8 = *(const u32x4_a2*)(bias_p + min(n0 + col0 + out_ch * 8, p.C_out - 8));
  unsigned bias_raw[CW / 64];
#pragma unroll
  for (int u = 0; u < CW / 64; ++u) bias_raw[u] = bias_p[min(n0 + wn * CW + 64 * u + lane, p.C_out - 1)];
  // (sum + bias) + addend, rounded
  auto finish = [&](int it, float (&v)[8]) __attribute__((always_inline)) {
    const u32x4 ad = p.addend ? addend_of(it) : u32x4{0u, 0u, 0u, 0u};
    u32x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float lo = v[2 * e] + (p.bias ? bf16_bits_to_float(bias8[e] & 0xffffu) : 0.f);
      float hi = v[2 * e + 1] + (p.bias ? bf16_bits_to_float(bias8[e] >> 16) : 0.f);
      if (p.addend) {
        lo += bf16_bits_to_float(ad[e] & 0xffffu);
        hi += bf16_bits_to_float(ad[e] >> 16);
      }
      bf16x2 pr;
      pr[0] = (__bf16)lo;
      pr[1] = (__bf16)hi;
      r[e] = __builtin_bit_cast(unsigned, pr);
    }
    __builtin_nontemporal_store(r, (u32x4*)(p.Out + out_offset(it)));
  };

  const int stages = __popcll(heads) * PARTS;
  if (stages == 0) {
    // no head of this token block is selected: the tile is addend + bias, straight from registers
    (void)fetch_addend();
#pragma unroll
    for (int it = 0; it < OUT_ITERS; ++it) {
      float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if (there(it)) finish(it, v);
    }
    return;
  }

  // scalar walks over the selected heads, PARTS stages per head, one for the weights and one for the tokens
  struct Walk {
    unsigned long long left;
    int part;
    __device__ __forceinline__ int next(int& part_out) {
      const int h = __builtin_ctzll(left);
      part_out = part;
      if (++part == PARTS) {
        part = 0;
        left &= left - 1ull;
      }
      return h;
    }
  };
  Walk ww = {heads, 0}, wx = {heads, 0};
  const size_t head_bytes = (size_t)p.L * (D * 2);
  auto w_src = [&]() {
    int part;
    const int h = ww.next(part);
    return sa_uniform_ptr(gW + ((size_t)h * D + (size_t)part * kStepK) * 2);
  };
  auto x_src = [&]() {
    int part;
    const int h = wx.next(part);
    return (size_t)sa_uniform_ptr((const char*)((size_t)h * head_bytes + (size_t)part * kRowB));
  };
  if constexpr (FLAGGED && !TWO) {
    st.run_short(smem, acc, stages, w_src, x_src, fetch_addend);
  } else if constexpr (kWhole) {
    st.run(smem, acc, stages, w_src, x_src, fetch_addend);
  } else {
    st.run(smem, acc, stages, w_src, x_src, []() { return 0; });
    (void)fetch_addend();
  }
  __syncthreads();   // every wave is done reading the stage buffers

  if (kWhole && p.addend) {
    // Epilogue with an addend: the accumulators (lane = token 32 * c + l32, registers = channels 32 * a + 8 * q4 + 4 * half
    // + 0..3 of the wave's corner) go to LDS as fp32 rows, 16-byte chunks permuted by the row so that the 32 tokens of an
    // access hit different banks, and come back as whole rows, to which a thread adds bias and addend.  Behind the arrival
    // of the addend there is nothing left but the store (33024 tokens, four heads per block, one term: 155 us; 164 with
    // the addend sent through LDS to the accumulators).
    auto chunk_at = [&](int row, int ch) -> char* { return smem + row * TN * 4 + ((ch ^ (row & 31)) * 16); };
#pragma unroll
    for (int a = 0; a < A; ++a)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
        for (int c = 0; c < C; ++c) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = acc[a][c][4 * q4 + e];
          *(f32x4*)chunk_at(wm * TW + 32 * c + l32, (wn * CW + 32 * a + 8 * q4) / 4 + half) = v;
        }
    sa_gemm::lds_barrier();
#pragma unroll
    for (int it = 0; it < OUT_ITERS; ++it) {
      const int row = it * RPI + out_row;
      const f32x4 v0 = *(const f32x4*)chunk_at(row, 2 * out_ch), v1 = *(const f32x4*)chunk_at(row, 2 * out_ch + 1);
      float v[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = v0[e];
        v[4 + e] = v1[e];
      }
      if (there(it)) finish(it, v);
    }
    return;
  }
  // Epilogue without an addend, and of 256 x 256 tiles, all in the wave's own piece of LDS (rows of CW bf16, 16-byte
  // chunks permuted by the row): the addend goes in as rows, comes out in the accumulators' layout, the sum (accumulator +
  // bias) + addend goes back rounded to the same place and leaves as rows.  LDS accesses of a wave execute in order, so
  // there is no barrier.
  constexpr int CHC = CW / 8, RPC = 64 / CHC;     // 16-byte pieces per row of the corner, rows per wave instruction
  const int c_row = lane / CHC, c_ch = lane % CHC;
  auto swizzle = [](int row) { return CHC == 16 ? (row & 15) : ((row >> 1) & 7); };
  char* const corner = smem + wave * TW * CW * 2;
  if constexpr (!kWhole) {
    if (p.addend) {
#pragma unroll
      for (int it = 0; it < OUT_ITERS; ++it) {
        const int row = it * RPC + c_row;
        if (there(it)) *(u32x4*)(corner + row * CW * 2 + ((c_ch ^ swizzle(row)) * 16)) = addend_of(it);
      }
    }
  }
  int bias_bits[CW / 64];
#pragma unroll
  for (int u = 0; u < CW / 64; ++u) bias_bits[u] = p.bias ? (int)(bias_raw[u] << 16) : 0;
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      float bv[4];                                 // channel 32 * a + 8 * q4 + 4 * half + e of the corner
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int ch = 32 * a + 8 * q4 + e;
        const int lo = __builtin_amdgcn_readlane(bias_bits[ch / 64], ch % 64), hi = __builtin_amdgcn_readlane(bias_bits[ch / 64], ch % 64 + 4);
        bv[e] = __builtin_bit_cast(float, half ? hi : lo);
      }
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const int row = 32 * c + l32;
        u32x2* const at = (u32x2*)(corner + row * CW * 2 + (((4 * a + q4) ^ swizzle(row)) * 16) + 8 * half);
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[a][c][4 * q4 + e] + bv[e];
        if (!kWhole && p.addend) {
          const u32x2 ad = *at;
          v[0] += bf16_bits_to_float(ad[0] & 0xffffu);
          v[1] += bf16_bits_to_float(ad[0] >> 16);
          v[2] += bf16_bits_to_float(ad[1] & 0xffffu);
          v[3] += bf16_bits_to_float(ad[1] >> 16);
        }
        bf16x2 lo, hi;
        lo[0] = (__bf16)v[0];
        lo[1] = (__bf16)v[1];
        hi[0] = (__bf16)v[2];
        hi[1] = (__bf16)v[3];
        u32x2 pk;
        pk[0] = __builtin_bit_cast(unsigned, lo);
        pk[1] = __builtin_bit_cast(unsigned, hi);
        *at = pk;
      }
    }
#pragma unroll
  for (int it = 0; it < TW / RPC; ++it) {
    const int row = it * RPC + c_row;
    const u32x4 v = *(const u32x4*)(corner + row * CW * 2 + ((c_ch ^ swizzle(row)) * 16));
    char* const out = p.Out + (((size_t)b * p.L + tok0 + wm * TW + row) * p.C_out + n0 + wn * CW + c_ch * 8) * 2;
    if (wm * TW + row < rows_valid && wn * CW + c_ch * 8 < cols_valid) __builtin_nontemporal_store(v, (u32x4*)out);
  }
}

template <int TM, int TN, int WM, int WN, int WB, int XB, int D, bool FLAGGED, bool TWO>
int launch_tiles(const GemmOParams& p, int B, hipStream_t stream) {
  constexpr size_t stage_lds = sa_gemm::Pipe<TN, TM, WN, WM, WB, XB>::kLdsBytes;
  constexpr size_t out_lds = (size_t)TM * TN * (TM * TN * 4 <= 160 * 1024 ? 4 : 2);   // the epilogue's rows
  constexpr size_t lds = stage_lds > out_lds ? stage_lds : out_lds;
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [] {
    attr_err = hipFuncSetAttribute((const void*)gemm_o_kernel<TM, TN, WM, WN, WB, XB, D, FLAGGED, TWO>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  });
  if (attr_err != hipSuccess)
    return sa_fail(SPARSE_ATTN_ERR_HIP, "hipFuncSetAttribute failed: %s", hipGetErrorString(attr_err));
  const int tiles = B * ((p.tok_end - p.tok_begin + TM - 1) / TM) * ((p.C_out + TN - 1) / TN);
  hipLaunchKernelGGL((gemm_o_kernel<TM, TN, WM, WN, WB, XB, D, FLAGGED, TWO>), dim3(tiles), dim3(WM * WN * 64), lds, stream, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return sa_fail(SPARSE_ATTN_ERR_HIP, "gemm_o launch failed: %s", hipGetErrorString(e));
  return 0;
}

// Which tile: without flags by the number of 128 x 128 tiles as in the query projection (33024 tokens, 24 heads of 128, 3072
// channels: 625 -> 512 us plain, 697 -> 602 with two terms); with flags one token block per tile, because the heads it
// visits are its own, and at least two workgroups per CU, because with few heads a tile is a chain of memory round trips
// (128 x 256 tiles, one per CU: 5 % slower at 90 % cached heads).
// Blocks of 64 tokens: tiles of 256 channels read the token rows half as often, tiles of 128 leave room for three
// workgroups per CU and fill the chip where tiles are few.  24 heads of 128, 3072 channels, us, 256 / 128 channels:
//   33024 tokens (6192 tiles of 256), one term:  2 heads per block 136 / 125, 4: 199 / 182, 8: 294 / 292, 24: 704 / 733
//   4608 tokens (864), no term:                  4 heads 27.3 / 28.0, 8: 42 / 45, 24: 101 / 112
//   1024 tokens (192), one term:                 4 heads 12.4 / 9.6, 24: 41 / 33
// So 128 channels up to 256 tiles (one per CU) and beyond 1280 (two and a half rounds of two per CU) where computed heads
// are selected, which are few; 256 channels in between and where cached heads are selected, which are many.  With two
// terms it is the addend that counts, not the heads: 256 channels beyond one per CU.
template <int D>
int launch(GemmOParams p, int B, int block_q, hipStream_t stream) {
  if (!p.flags) {
    const int tok = p.tok_end - p.tok_begin;
    const long long units = (long long)B * ((tok + 127) / 128) * (p.C_out / 128);
    if (units <= kCus) return launch_tiles<128, 128, 2, 2, 2, 3, D, false, true>(p, B, stream);
    if (units <= 2 * kCus) return launch_tiles<256, 128, 4, 2, 3, 3, D, false, true>(p, B, stream);
    const int n_col = (p.C_out + 255) / 256, n_tok = (tok + 255) / 256;
    const long long tiles = (long long)B * n_tok * n_col, full = tiles / kCus * kCus;
    const int keep = (int)(full / ((long long)B * n_col));
    if (tiles > full && tiles - full <= kCus / 2 && keep > 0) {
      GemmOParams rest = p;
      p.tok_end = rest.tok_begin = p.tok_begin + keep * 256;
      if (int rc = launch_tiles<256, 256, 4, 2, 2, 3, D, false, true>(p, B, stream)) return rc;
      return launch<D>(rest, B, block_q, stream);
    }
    return launch_tiles<256, 256, 4, 2, 2, 3, D, false, true>(p, B, stream);
  }
  if (block_q == 128) return launch_tiles<128, 128, 2, 2, 2, 3, D, true, true>(p, B, stream);
  const long long tiles = (long long)B * ((p.L + 63) / 64) * ((p.C_out + 255) / 256);
  if (p.n_terms > 1) {
    if (tiles <= kCus) return launch_tiles<64, 128, 1, 2, 2, 3, D, true, true>(p, B, stream);
    return launch_tiles<64, 256, 1, 4, 2, 2, D, true, true>(p, B, stream);
  }
  if (tiles <= kCus || (tiles > 5 * kCus && !p.select)) return launch_tiles<64, 128, 1, 2, 2, 2, D, true, false>(p, B, stream);
  return launch_tiles<64, 256, 1, 4, 2, 2, D, true, true>(p, B, stream);
}

bool ranges_overlap(const void* a, size_t na, const void* b, size_t nb) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + nb && y < x + na;
}

}  // namespace

namespace {

int gemm_o_run(const void* O, const void* W, const void* bias, const uint8_t* cache_flags, int select_cached,
               const void* addend, const void* const* terms, const float* coef, int n_terms, void* Out, int B, int H,
               int L, int D, int C_out, int block_q, hipStream_t stream) {
  if (B <= 0 || H <= 0 || L <= 0 || D <= 0 || C_out <= 0 || block_q <= 0)
    return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_o: sizes must be positive (B=%d H=%d L=%d D=%d C_out=%d block_q=%d)",
                   B, H, L, D, C_out, block_q);
  if (select_cached != 0 && select_cached != 1)
    return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_o: select_cached must be 0 or 1 (got %d)", select_cached);
  if ((D != 64 && D != 128) || (block_q != 64 && block_q != 128))
    return sa_fail(SPARSE_ATTN_ERR_UNSUPPORTED, "gemm_o: D and block_q must be 64 or 128 (got %d, %d)", D, block_q);
  if (H > 64) return sa_fail(SPARSE_ATTN_ERR_UNSUPPORTED, "gemm_o: at most 64 heads (got %d)", H);
  if (C_out % kBN)
    return sa_fail(SPARSE_ATTN_ERR_UNSUPPORTED, "gemm_o: C_out=%d must be a multiple of %d", C_out, kBN);
  if ((long long)kBN * H * D * 2 >= (1LL << 31)) return sa_fail(SPARSE_ATTN_ERR_UNSUPPORTED, "gemm_o: H*D too large");
  const int tq = (L + block_q - 1) / block_q;      // a short last block counts as a block
  const long long tiles = (long long)B * tq * (C_out / kBN);
  if (tiles > 0x3fffffffLL) return sa_fail(SPARSE_ATTN_ERR_UNSUPPORTED, "gemm_o: too many tiles (%lld)", tiles);
  if (!O || !W || !Out) return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_o: O, W and Out must not be NULL");
  if (((uintptr_t)O | (uintptr_t)W | (uintptr_t)Out | (uintptr_t)addend) & 15)
    return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_o: O, W, addend and Out must be 16-byte aligned");
  const size_t ob = (size_t)B * H * L * D * 2, wb = (size_t)C_out * H * D * 2, outb = (size_t)B * L * C_out * 2;
  if (ranges_overlap(Out, outb, O, ob) || ranges_overlap(Out, outb, W, wb))
    return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_o: Out must not overlap O or W");
  if (addend && addend != Out && ranges_overlap(Out, outb, addend, outb))
    return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_o: addend must be Out itself or must not overlap Out");

  GemmOParams p;
  p.O = (const char*)O;
  p.W = (const char*)W;
  p.bias = (const uint16_t*)bias;
  p.flags = cache_flags;
  p.addend = (const char*)addend;
  p.Out = (char*)Out;
  p.H = H;
  p.L = L;
  p.tok_begin = 0;
  p.tok_end = L;
  p.C_out = C_out;
  p.select = select_cached;
  p.n_terms = 0;
  for (int d = 0; d < kMaxTerms; ++d) p.coef[d] = 0.f;
  for (int d = 0; d + 1 < kMaxTerms; ++d) p.term[d] = nullptr;
  if (terms) {
    if (n_terms < 1 || n_terms > kMaxTerms)
      return sa_fail(SPARSE_ATTN_ERR_UNSUPPORTED, "gemm_o: n_terms=%d must be between 1 and %d", n_terms, kMaxTerms);
    if (!coef) return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_o: coef must not be NULL");
    for (int d = 0; d < n_terms; ++d) {
      if (!terms[d]) return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_o: terms[%d] must not be NULL", d);
      if ((uintptr_t)terms[d] & 15) return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_o: terms[%d] must be 16-byte aligned", d);
      if (terms[d] != Out && ranges_overlap(Out, outb, terms[d], outb))
        return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_o: terms[%d] must be Out itself or must not overlap Out", d);
      if (!(coef[d] == coef[d]) || coef[d] - coef[d] != 0.f)
        return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_o: coef[%d] must be finite", d);
    }
    p.addend = (const char*)terms[0];
    if (!(n_terms == 1 && coef[0] == 1.0f)) {      // one term with weight 1 is the plain addend
      p.n_terms = n_terms;
      for (int d = 0; d < n_terms; ++d) p.coef[d] = coef[d];
      for (int d = 1; d < n_terms; ++d) p.term[d - 1] = (const char*)terms[d];
    }
  }
  return D == 128 ? launch<128>(p, B, block_q, stream) : launch<64>(p, B, block_q, stream);
}

}  // namespace

extern "C" {

int sparse_gemm_o_stream(const void* O, const void* W, const void* bias, const uint8_t* cache_flags,
                         int select_cached, const void* addend, void* Out, int B, int H, int L, int D, int C_out,
                         int block_q, void* hip_stream) {
  return gemm_o_run(O, W, bias, cache_flags, select_cached, addend, nullptr, nullptr, 0, Out, B, H, L, D, C_out, block_q,
                    (hipStream_t)hip_stream);
}

int sparse_gemm_o(const void* O, const void* W, const void* bias, const uint8_t* cache_flags, int select_cached,
                  const void* addend, void* Out, int B, int H, int L, int D, int C_out, int block_q) {
  return sparse_gemm_o_stream(O, W, bias, cache_flags, select_cached, addend, Out, B, H, L, D, C_out, block_q, nullptr);
}

int sparse_gemm_o_reuse(const void* O, const void* W, const void* bias, const uint8_t* cache_flags,
                        const void* const* terms, const float* coef, int n_terms, void* Out, int B, int H, int L, int D,
                        int C_out, int block_q, void* hip_stream) {
  if (!terms) return sa_fail(SPARSE_ATTN_ERR_INVALID, "gemm_o: terms must not be NULL");
  return gemm_o_run(O, W, bias, cache_flags, 0, nullptr, terms, coef, n_terms, Out, B, H, L, D, C_out, block_q,
                    (hipStream_t)hip_stream);
}

}  // extern "C"
