// Shared between the translation units of the library (not part of the public ABI).
#ifndef SPARSE_ATTN_INTERNAL_H
#define SPARSE_ATTN_INTERNAL_H

#include <hip/hip_runtime.h>

#include <type_traits>

// Records a printf-style message for sparse_attn_last_error() on the calling thread and returns `code`.
int sa_fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));

// The library's scratch buffer of the current device and `stream`, grown (with a stream synchronisation) to at
// least `need` bytes.  Every entry point that needs scratch memory shares it: work on one stream runs in
// order, and no entry point keeps anything in it between calls.
int sa_get_scratch(size_t need, hipStream_t stream, void** out);

// Direct-to-LDS load: every lane fetches 16 bytes from gbase (wave-uniform) + lane_off, the wave's
// 1 KiB lands at consecutive LDS addresses starting at the wave-uniform `lds_addr`.  Written as
// inline assembly so that the compiler does not serialise later LDS reads of the OTHER buffer
// behind these loads (it cannot tell the two buffers apart); the kernels wait for them themselves
// (s_waitcnt vmcnt(0) + barrier) before the buffer is read.  A scalar write of M0 and the load that takes its LDS address from
// it need one wait state between them, which the compiler keeps for its own instructions but not inside a statement.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void sa_load_to_lds_16B(const char* gbase, unsigned lane_off, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds_addr), "v"(lane_off), "s"(gbase)
               : "memory", "m0");
}
#pragma clang diagnostic pop

// A wave-uniform pointer that the compiler may have left in vector registers, moved to scalar registers.
__device__ __forceinline__ const char* sa_uniform_ptr(const char* ptr) {
  const unsigned long long v = (unsigned long long)ptr;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return (const char*)(((unsigned long long)hi << 32) | lo);
}

// s_waitcnt vmcnt(0) only: expcnt and lgkmcnt fields left at their maxima
__device__ __forceinline__ void sa_wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }
// s_waitcnt vmcnt(N): at most the N newest vector-memory requests of the wave are still outstanding (loads
// return in order).  The six-bit count is split over bits 3:0 and 15:14 of the immediate.
template <int N>
__device__ __forceinline__ void sa_wait_vmem_but() {
  static_assert(N >= 0 && N < 64, "vmcnt is a six-bit counter");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// ---------------------------------------------------------------------------------------
// Reduction loop of the two projection kernels (query and output projection).
//
// Both compute a transposed product C^T[n][token] = sum_k W[n][k] X[token][k] with v_mfma_f32_32x32x16_bf16 (A = weight
// rows, B = token rows, both k-contiguous) and stream the operands through LDS, kStepK reduction channels per stage,
// rows of kRowB bytes.  The 16-byte chunks of a row are permuted by row_swizzle so that the operand reads of a wave
// spread over all banks; a direct-to-LDS load writes consecutive LDS, so the permutation is applied to the global
// address each lane fetches.
// ---------------------------------------------------------------------------------------
namespace sa_gemm {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int kCus = 256;           // compute units of the MI355X: what the choice of a tile counts rounds with
constexpr int kStepK = 64;          // reduction channels per LDS stage
constexpr int kRowB = kStepK * 2;   // bytes per tile row in LDS

// 16-byte chunk permutation of a 128-byte tile row (two rows share a 256-byte bank line)
__device__ __forceinline__ int row_swizzle(int row) { return (row >> 1) & 7; }

// Barrier that waits for this wave's LDS traffic only; __syncthreads() would also wait for its outstanding loads.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The reduction loop on a tile of TN weight rows x TM token rows, WN x WM waves, every wave a corner of TN / WN
// channels x TM / WM tokens (kA x kC accumulators of 32 x 32).  A stage is kStepK channels; the weight rows have WB
// buffers in LDS, the token rows XB (2 or 3 each, XB >= WB).  LDS: the weight buffers, then the token buffers.
// Per stage s and wave, ks = 16-channel step:
//     ks 0 | operands of ks 1 are read           | MFMAs, between them requests: weights of stage s + WB - 1, 2nd half
//     ks 1 | operands of ks 2                    | ... token rows of stage s + XB - 1, 1st half
//     ks 2 | operands of ks 3                    | ... 2nd half
//     stage s + 1 has landed (everything but what belongs to later stages), all waves' reads have returned: barrier
//     ks 3 | operands of ks 0 of stage s + 1     | ... weights of stage s + WB, 1st half
// (XB = 2: the token rows of stage s + 2 go out like the weights, the first half in ks 3, in front of theirs, the second in ks
// 0 of the next stage.  In ks 1 and 2, half a stage behind the barrier that frees their buffer, they arrive late: query
// projection, 9001 tokens, 24 heads of 64, 90 % cached 25.0 -> 22.6 us; all of them in ks 3 crowds that step: 4608 tokens, 64
// heads of 64, half cached, blocks of 128 tokens 90.3 -> 94.6.)
// so a step's operands are on their way while the previous step's MFMAs run, across the stage boundary too; the
// requests go out one at a time behind an MFMA (in a burst they keep the wave from issuing the next one).
// Buffer safety: the weights requested in ks 3 of stage s (and ks 0 of the next) overwrite those of stage s, the token
// rows requested in ks 1 and 2 those of stage s - 1 (XB = 2: ks 3 and the next ks 0, of stage s); all waves' reads of a stage have returned
// at the barrier inside it.
template <int TN, int TM, int WN, int WM, int WB, int XB>
struct Pipe {
  static constexpr int kWaves = WN * WM;
  static constexpr int kA = TN / WN / 32, kC = TM / WM / 32;
  static constexpr int kWStage = TN * kRowB, kXStage = TM * kRowB;
  static constexpr int kX0 = WB * kWStage;                       // first token buffer
  static constexpr int kLdsBytes = WB * kWStage + XB * kXStage;
  static constexpr int kWLoad = kWStage / 1024 / kWaves;         // direct-to-LDS wave instructions per stage and wave
  static constexpr int kXLoad = kXStage / 1024 / kWaves;         // (8 rows each)
  static constexpr int kAhead = (WB == 3 ? kWLoad : 0) + (XB == 3 ? kXLoad : 0);   // of these requested two stages ahead
  static constexpr int kSteps = kStepK / 16;
  static_assert((kWStage / 1024) % kWaves == 0 && (kXStage / 1024) % kWaves == 0, "stage loads must split evenly over the waves");
  static_assert(WB >= 2 && XB >= WB && XB <= 3, "two or three buffers");

  unsigned w_goff[kWLoad], x_goff[kXLoad];   // per-lane global offsets of this wave's stage loads
  const char* x_base[kXLoad];                // (wave-uniform) what the token offsets start from
  int w_off[kSteps], x_off[kSteps];          // per-lane LDS offsets of the operand reads, k-step ks, buffer 0
  unsigned lds_base;
  int wave;

  // Tile row of lane `lane` in the wave's u-th load of a stage.
  __device__ __forceinline__ static int load_row(int wave, int lane, int u) { return (wave + u * kWaves) * 8 + lane / 8; }

  // wn / wm: this wave's corner; w_pitch: bytes between weight rows in memory.  Weight rows from w_rows_valid on do
  // not exist: their loads re-read the last row that does, and the caller never stores their results.  The token rows
  // are the caller's: set_x_rows() for every u.
  __device__ __forceinline__ void init(unsigned lds_base_, int wave_, int lane, int wn, int wm, size_t w_pitch, int w_rows_valid) {
    lds_base = lds_base_;
    wave = wave_;
    const int l32 = lane & 31, half = lane >> 5;
#pragma unroll
    for (int u = 0; u < kWLoad; ++u) {
      const int r = load_row(wave, lane, u);
      w_goff[u] = (unsigned)(min(r, w_rows_valid - 1) * w_pitch + (((lane % 8) ^ row_swizzle(r)) * 16));
    }
#pragma unroll
    for (int ks = 0; ks < kSteps; ++ks) {
      const int o = l32 * kRowB + (((2 * ks + half) ^ row_swizzle(l32)) * 16);
      w_off[ks] = wn * (TN / WN) * kRowB + o;
      x_off[ks] = kX0 + wm * (TM / WM) * kRowB + o;
    }
  }
  // The wave's u-th load reads memory row `row` (per lane) of the rows that start at `base` (wave-uniform).
  __device__ __forceinline__ void set_x_rows(int u, const char* base, int row, size_t pitch, int lane) {
    x_base[u] = base;
    x_goff[u] = (unsigned)(row * pitch + (((lane % 8) ^ row_swizzle(load_row(wave, lane, u))) * 16));
  }

  // requests lo .. hi - 1 of this wave's kWLoad / kXLoad of a stage
  __device__ __forceinline__ void issue_w(const char* src, int buf, int lo, int hi) const {
#pragma unroll
    for (int u = lo; u < hi; ++u)
      sa_load_to_lds_16B(src, w_goff[u], lds_base + (unsigned)(buf * kWStage + (wave + u * kWaves) * 1024));
  }
  __device__ __forceinline__ void issue_x(size_t k_off, int buf, int lo, int hi) const {
#pragma unroll
    for (int u = lo; u < hi; ++u)
      sa_load_to_lds_16B(x_base[u] + k_off, x_goff[u], lds_base + (unsigned)(kX0 + buf * kXStage + (wave + u * kWaves) * 1024));
  }

  // w_src / x_src: functors, called once per stage and in order: the (wave-uniform) address of the first weight row's
  // channels of the next stage, and the offset of its token channels from x_base.  On return every wave has read its
  // last operands; LDS may be written after a barrier.
  // extra: called once, when the last stage has been requested and one to two stages of MFMAs are still to come, for
  // plain loads whose results are used behind the loop; it returns a number of load instructions that it has
  // certainly issued (loads return in order: the wait for the last stage may leave that many out).
  template <class WSrc, class XSrc, class Extra>
  __device__ __forceinline__ void run(const char* smem, f32x16 (&acc)[kA][kC], int stages, WSrc&& w_src, XSrc&& x_src,
                                      Extra&& extra) const {
    bf16x8 wa[2][kA], xb[2][kC];
    auto read = [&](auto ks_c, const char* wbase, const char* xbase) __attribute__((always_inline)) {
      constexpr int ks = decltype(ks_c)::value;
#pragma unroll
      for (int c = 0; c < kC; ++c) xb[ks & 1][c] = *(const bf16x8*)(xbase + c * 32 * kRowB + x_off[ks]);
#pragma unroll
      for (int a = 0; a < kA; ++a) wa[ks & 1][a] = *(const bf16x8*)(wbase + a * 32 * kRowB + w_off[ks]);
    };
    // the MFMAs of a step with n requests spread between them: ask(j) makes the j-th
    auto mfma = [&](auto ks_c, auto n_c, auto&& ask) __attribute__((always_inline)) {
      constexpr int ks = decltype(ks_c)::value, n = decltype(n_c)::value;
      int j = 0;
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int m = 0; m < kA * kC; ++m) {
        const int a = m / kC, c = m % kC;
        acc[a][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[ks & 1][a], xb[ks & 1][c], acc[a][c], 0, 0, 0);
        if (j < n && (m + 1) * n >= (j + 1) * kA * kC - n / 2) {
          __builtin_amdgcn_sched_barrier(0);
          ask(j++);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (; j < n; ++j) ask(j);
    };
    using K0 = std::integral_constant<int, 0>;
    using K1 = std::integral_constant<int, 1>;
    using K2 = std::integral_constant<int, 2>;
    using K3 = std::integral_constant<int, 3>;
    static_assert(kSteps == 4, "the loop below is written for four 16-channel steps");

    constexpr int w1 = kWLoad / 2, w2 = kWLoad - w1, x1 = kXLoad / 2, x2 = kXLoad - x1;   // halves of a stage's requests
    const char* w_at = w_src();
    issue_w(w_at, 0, 0, kWLoad);
    issue_x(x_src(), 0, 0, kXLoad);
    if (WB == 3 && stages > 1) issue_w(w_src(), 1, 0, kWLoad);
    size_t x_next = 0;                           // XB = 2: the token channels that the next ks 0 asks for the rest of
    if (stages > 1) {
      x_next = x_src();
      issue_x(x_next, 1, 0, XB == 3 ? kXLoad : x1);
    }
    if (stages >= WB) {
      w_at = w_src();
      issue_w(w_at, WB - 1, 0, w1);
    }
    if (stages >= 3)
      sa_wait_vmem_but<(WB - 2) * kWLoad + (XB == 3 ? kXLoad : x1) + w1>();
    else
      sa_wait_vmem();
    lds_barrier();
    int wbuf = 0, xbuf = 0;                      // buffers of this stage
    const char* wb = smem;
    const char* xb0 = smem;
    read(K0{}, wb, xb0);
    // nothing is pending on the way into the loop (s_waitcnt lgkmcnt(0)): otherwise the compiler cannot tell the reads
    // of one step from those of the next and waits for both before the first MFMA of every stage
    __builtin_amdgcn_s_waitcnt(0xC07F);
    // one stage; whether there is a next stage, one after it, and weights to ask for in ks 3 are compile-time matters,
    // so that the steady state has no branch in it (a branch between the operand reads and the MFMAs makes the
    // compiler wait for all reads at once)
    auto stage = [&](auto more1_c, auto more2_c, auto ask_w_c) __attribute__((always_inline)) {
      constexpr bool more1 = decltype(more1_c)::value, more2 = decltype(more2_c)::value, ask_w = decltype(ask_w_c)::value;
      constexpr bool ask_w2 = WB == 3 ? more2 : more1, ask_x = XB == 3 && more2, ask_x2 = XB == 2 && more2, ask_x1 = XB == 2 && more1;
      const int w_free = wbuf == 0 ? WB - 1 : wbuf - 1, x_free = xbuf == 0 ? XB - 1 : xbuf - 1;
      read(K1{}, wb, xb0);
      mfma(K0{}, std::integral_constant<int, (ask_x1 ? x2 : 0) + (ask_w2 ? w2 : 0)>{}, [&](int j) {
        if (ask_x1 && j < x2)
          issue_x(x_next, x_free, x1 + j, x1 + j + 1);
        else
          issue_w(w_at, w_free, w1 + j - (ask_x1 ? x2 : 0), w1 + j - (ask_x1 ? x2 : 0) + 1);
      });
      int behind = 0;
      if constexpr (more1 && !more2) {
        behind = extra();
        asm volatile("" ::: "memory");             // none of its loads moves down past the wait that counts on them
      }
      size_t x_at = 0;
      if constexpr (ask_x) x_at = x_src();
      read(K2{}, wb, xb0);
      mfma(K1{}, std::integral_constant<int, ask_x ? x1 : 0>{}, [&](int j) { issue_x(x_at, x_free, j, j + 1); });
      read(K3{}, wb, xb0);
      mfma(K2{}, std::integral_constant<int, ask_x ? x2 : 0>{}, [&](int j) { issue_x(x_at, x_free, x1 + j, x1 + j + 1); });
      const int w_done = wbuf, x_done = xbuf;
      if constexpr (more1) {
        if constexpr (more2)
          sa_wait_vmem_but<kAhead>();
        else if (behind >= 16)
          sa_wait_vmem_but<16>();
        else if (behind >= 8)
          sa_wait_vmem_but<8>();
        else
          sa_wait_vmem();
        lds_barrier();
        wbuf = wbuf == WB - 1 ? 0 : wbuf + 1;
        xbuf = xbuf == XB - 1 ? 0 : xbuf + 1;
        wb = smem + wbuf * kWStage;
        xb0 = smem + xbuf * kXStage;
        read(K0{}, wb, xb0);
        if constexpr (ask_x2) x_next = x_src();
        if constexpr (ask_w) w_at = w_src();
      }
      mfma(K3{}, std::integral_constant<int, (ask_x2 ? x1 : 0) + (ask_w ? w1 : 0)>{}, [&](int j) {
        if (ask_x2 && j < x1)
          issue_x(x_next, x_done, j, j + 1);
        else
          issue_w(w_at, w_done, j - (ask_x2 ? x1 : 0), j - (ask_x2 ? x1 : 0) + 1);
      });
    };
    using T = std::true_type;
    using F = std::false_type;
    int left = stages;                           // stages left, this one included: s + 3 < stages <=> left > 3
    for (; left > 3; --left) stage(T{}, T{}, T{});
    if (left == 3) {
      stage(T{}, T{}, std::integral_constant<bool, WB == 2>{});
      --left;
    }
    if (left == 2)
      stage(T{}, F{}, F{});
    else
      (void)extra();
    stage(F{}, F{}, F{});
  }

  // The loop for few stages (the heads that the flags of a token block select).  There a tile is a chain of round trips
  // to memory, and what counts is that a stage is requested early: all of it in one go, as soon as the barrier has freed
  // its buffers (output projection, 64 x 128 tiles, 33024 tokens, two heads per block: 99 us, 102 with run(); 1024
  // tokens, 24 heads: 32 against 35).
  // early: called behind the first stage's requests for plain loads whose results are used behind the loop; it returns
  // 8 if it has certainly issued that many load instructions, else 0 (loads return in order: the wait for the first stage
  // may leave them out).
  template <class WSrc, class XSrc, class Early>
  __device__ __forceinline__ void run_short(const char* smem, f32x16 (&acc)[kA][kC], int stages, WSrc&& w_src, XSrc&& x_src,
                                            Early&& early) const {
    static_assert(WB == 2 && XB == 2, "two buffers");
    auto issue = [&](auto buf_c) __attribute__((always_inline)) {
      issue_w(w_src(), decltype(buf_c)::value, 0, kWLoad);
      issue_x(x_src(), decltype(buf_c)::value, 0, kXLoad);
    };
    using B0 = std::integral_constant<int, 0>;
    using B1 = std::integral_constant<int, 1>;
    int left = stages;
    bool first = true;
    int early_loads = 0;
    auto step = [&](auto buf_c, auto other_c) __attribute__((always_inline)) {
      constexpr int buf = decltype(buf_c)::value;
      if (first && early_loads == 8)
        sa_wait_vmem_but<8>();
      else
        sa_wait_vmem();
      first = false;
      lds_barrier();                               // this stage has landed for every wave; the other buffers are free
      if (--left > 0) issue(other_c);
      bf16x8 wa[kSteps][kA], xb[kSteps][kC];
#pragma unroll
      for (int ks = 0; ks < kSteps; ++ks) {
#pragma unroll
        for (int a = 0; a < kA; ++a) wa[ks][a] = *(const bf16x8*)(smem + buf * kWStage + a * 32 * kRowB + w_off[ks]);
#pragma unroll
        for (int c = 0; c < kC; ++c) xb[ks][c] = *(const bf16x8*)(smem + buf * kXStage + c * 32 * kRowB + x_off[ks]);
      }
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int ks = 0; ks < kSteps; ++ks)
#pragma unroll
        for (int a = 0; a < kA; ++a)
#pragma unroll
          for (int c = 0; c < kC; ++c) acc[a][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[ks][a], xb[ks][c], acc[a][c], 0, 0, 0);
      __builtin_amdgcn_s_setprio(0);
    };
    issue(B0{});
    early_loads = early();
    asm volatile("" ::: "memory");                 // none of its loads moves down past the wait that counts on them
    while (left > 0) {
      step(B0{}, B1{});
      if (left == 0) break;
      step(B1{}, B0{});
    }
  }
};

}  // namespace sa_gemm

#endif
