// Expert FFN products (bf16) for steps with few rows per expert: more than the matrix-vector kernels serve, fewer than
// fill the grouped GEMM's 256-row tiles (a serving batch that generates, Section 3.3).
//
//   out[r, n] = epilogue( sum_k act[r, k] * W_e[n, k] )      for the rows r of every expert
//
// The product's time is the time to stream the activated experts' weights once.  The 256 x 256 tiles of the grouped GEMM
// have one 64 KB stage in flight per CU, half of it rows that are not there, and their number is too small for the chip
// when the feature count is: 8 experts x 4096 features are 128 tiles for 256 CUs.  Here a workgroup owns 64 to 256 weight
// rows and 32 to 192 rows of one expert and requests the stages of all but one of its three to five LDS buffers (64 values of the
// contraction index each) ahead, though the queue drains once per 24 steps (see the K loop): weights and
// rows go from global memory straight into LDS, swizzled like the grouped GEMM's, one barrier per stage.  A wavefront multiplies blocks of 16 weight rows by blocks of 16 rows
// (v_mfma_f32_16x16x32_bf16, weights as the first operand: a lane ends up with four consecutive features of one row).
// SwiGLU: half of the weight rows are the gate's and half the up projection's; a block of 16 is eight and eight of the
// same features.
#include <type_traits>
#include <utility>
#include "moesys_internal.h"
#include "phi_table.h"
#include "row_tiles.h"
#include "wave_util.h"

namespace moesys {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

enum StreamEpi { ST_GELU = 0, ST_SWIGLU = 1, ST_BIAS = 2, ST_COMBINE = 3 };

constexpr int ST_KS = 64;     // values of the contraction index per stage: LDS rows of 128 bytes, eight 16-byte chunks

// NWF x NWM wavefronts, each FB blocks of 16 weight rows x RB blocks of 16 rows; stages of weights, and of rows if fewer
template <int NWF_, int NWM_, int FB_, int RB_, int STAGES_, int ROW_STAGES_ = STAGES_>
struct StreamShape {
  static constexpr int NWF = NWF_, NWM = NWM_, FB = FB_, RB = RB_, STAGES = STAGES_, ROW_STAGES = ROW_STAGES_;
  static constexpr int WAVES = NWF * NWM, WROWS = NWF * FB * 16, TM = NWM * RB * 16;
};

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}
__device__ __forceinline__ float lo16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi16(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float gelu_exact(float u) { return 0.5f * u * erfcf(-u * 0.70710678118654752f); }
constexpr int LOAD_NT = 2;  // cache policy of a buffer load: non-temporal
// s_waitcnt operand: at most n vector memory operations and no LDS operation in flight
constexpr int wait_vm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0070; }

#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t stream_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
#endif

// f(integral_constant<int, 0>{}, ..., integral_constant<int, N - 1>{})
template <typename F, int... I>
__device__ __forceinline__ bool unrolled_of(F& f, std::integer_sequence<int, I...>) { return f(std::integral_constant<int, I>{}...); }
template <int N, typename F>
__device__ __forceinline__ bool unrolled(F& f) { return unrolled_of(f, std::make_integer_sequence<int, N>{}); }

// NT: the call's weights exceed the last-level cache (weights_exceed_cache)
template <int EPI, bool GATHER, bool NT, typename S>
__global__ __launch_bounds__(S::WAVES * 64) void expert_stream_kernel(
    const uint16_t* __restrict__ act, const uint16_t* __restrict__ wa, const uint16_t* __restrict__ wb,
    const uint16_t* __restrict__ bias, const int32_t* __restrict__ offsets, uint16_t* out,
    const int32_t* __restrict__ row_map, const float* __restrict__ gate_w, const uint16_t* residual,
    const int32_t* __restrict__ a2r, const int64_t* __restrict__ eoff, int32_t* __restrict__ clear_ctr, int T, int E, int N, int K, int n_tiles) {
#if defined(__HIP_DEVICE_COMPILE__)  // (buffer descriptors are device-only types)
  constexpr int TM = S::TM, STAGES = S::STAGES, ROW_STAGES = S::ROW_STAGES, ST_WAVES = S::WAVES, FB = S::FB, RB = S::RB;
  constexpr int OUTF = EPI == ST_SWIGLU ? S::WROWS / 2 : S::WROWS;  // output features per workgroup
  constexpr int W_BYTES = S::WROWS * 128, A_BYTES = TM * 128;
  constexpr bool SPLIT = ROW_STAGES != STAGES;  // the shape for 97 to 160 rows
  constexpr int A_BLKS = TM / 8;  // blocks of eight rows, one load each
  constexpr int W_LOADS = W_BYTES / 1024 / ST_WAVES, A_LOADS = A_BLKS / ST_WAVES, LOADS = W_LOADS + A_LOADS;
  static_assert(W_BYTES % (1024 * ST_WAVES) == 0 && A_BLKS % ST_WAVES == 0, "whole loads of 8 rows per wavefront");
  static_assert(STAGES >= 3 && STAGES <= 5 && (ROW_STAGES == STAGES || (STAGES == 3 && ROW_STAGES == 2)), "the K loop below");
  // one array per stage: the compiler can then tell the stages being filled from the one being read
  __shared__ __attribute__((aligned(1024))) unsigned char w0[W_BYTES], a0[A_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char w1[W_BYTES], a1[A_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char w2[W_BYTES], a2[ROW_STAGES > 2 ? A_BYTES : 16];
  __shared__ __attribute__((aligned(1024))) unsigned char w3[STAGES > 3 ? W_BYTES : 16], a3[ROW_STAGES > 3 ? A_BYTES : 16];
  __shared__ __attribute__((aligned(1024))) unsigned char w4[STAGES > 4 ? W_BYTES : 16], a4[ROW_STAGES > 4 ? A_BYTES : 16];
  // GELU: by the exact function for a few elements per lane, by the table for many: filled while the first stages are on their way
  // where the LDS has room for it beside them, else in the first stage's buffer behind the K loop.  Measured on MI355X, whole layers
  // (us, behind the loop / beside the stages): 64 experts 1024 x 4096, 128 rows 307.5 / 303.0; 64 of 1600 x 6144, 88 rows 624 / 618;
  // 32 of 1024 x 2048, 94 rows 106.8 / 105.3.
  constexpr bool TABLE = EPI == ST_GELU && FB * RB >= 8;
  constexpr bool OWN_TABLE = TABLE && STAGES * W_BYTES + ROW_STAGES * A_BYTES + PHI_N * 8 <= 159 * 1024;
  static_assert(PHI_N * 8 <= W_BYTES, "the table fits a stage of weights");
  __shared__ __attribute__((aligned(16))) unsigned char table[OWN_TABLE ? PHI_N * 8 : 16];
  if (clear_ctr && blockIdx.x == 0 && threadIdx.x < 8) clear_ctr[threadIdx.x] = 0;  // (a grouped GEMM may run next)
  RowTile t;
  const int kept = EPI == ST_COMBINE ? offsets[E] : 0;
  // SwiGLU on 64x32, the XCDs' eighths a multiple of 16 MB apart (as the two matrices then are as well): in step they meet on the same memory
  // channels, the more so the longer they run without a drain (8 experts 4096 x 14336, 12 and 24 rows: 485 us a layer, with passes of four steps
  // 462).  MI355X, whole layers of 1 to 24 rows against eighths that all start in front: 4096 values 1.048 over 55, up to 1.152 (16 experts
  // x 2048: 166 / 191), 2048 1.018 over 54, 12288 1.037 over 10, 1024, 5120, 6144 and 8192 1.000 to 1.010.  Where the eighths lie otherwise the
  // shift loses as often (a multiple of 4 MB, 4096 values 0.972 over 40), and GELU, the second product and the larger shapes measured 0.99 to
  // 1.01 with it.  7, 13, 21 and 29 tiles are within 1 %, but 21 at 12288 values 0.97.
  constexpr int SHIFT = EPI == ST_SWIGLU && TM == 32 ? 13 : 0;
  const bool have = find_row_tile<TM, 0, SHIFT>(offsets, E, n_tiles, t, (uint32_t)(OUTF * K * 2));
  if constexpr (EPI == ST_COMBINE) fill_rowless_tokens<ST_WAVES>(a2r, kept, T, N, residual, out);
  if (!have) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // a feature count that is no multiple of the tile: the last tile starts at N - OUTF and leaves to the one before what is its
  const int n0 = min(t.nt * OUTF, N - OUTF);
  const int KT = K / ST_KS;
  const int64_t wbase = (eoff ? eoff[t.expert] : (int64_t)t.expert * N * K) + (int64_t)n0 * K;

  // ---- loads: one instruction moves 8 rows of 128 bytes; lane l lands at row l / 8, physical chunk l mod 8 of the eight
  // rows, which holds the logical chunk (l mod 8) ^ key, key = (row / 2) mod 8.  SwiGLU: LDS rows 16 w .. 16 w + 7 are the
  // gate rows of features 8 w .. 8 w + 7, the eight after them their up rows.
  auto block = [&](int i) { return (i < W_LOADS ? i : i - W_LOADS) * ST_WAVES + wave; };
  const int k2 = K * 2;  // bytes of a row
  int voff[LOADS];
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int blk = block(i);  // which eight LDS rows
    const int row = blk * 8 + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
    int r = row;
    if (i < W_LOADS) {
      if (EPI == ST_SWIGLU) r = (blk >> 1) * 8 + (lane >> 3);
    } else {
      r = min(row, t.rows - 1);  // (rows past the last re-read it; their results are not stored)
      if (GATHER) {
        r = row_map[t.row0 + r];
        while (r >= T) r -= T;  // assignment id j*T + t -> token (j < k <= 8)
      }
    }
    voff[i] = r * k2 + chunk * 16;
    // (a third of this shape's rows may be missing: out of range, they read as zero without going to memory)
    if (SPLIT && i >= W_LOADS && row >= t.rows) voff[i] = 0x7fffffff;
  }
  const uint16_t* a_ptr = GATHER ? act : act + (int64_t)t.row0 * K;
  const uint32_t a_bytes = (uint32_t)(GATHER ? T : t.rows) * (uint32_t)k2, w_bytes = (uint32_t)OUTF * (uint32_t)k2;
  // Weights that only this workgroup reads pass the caches by where the call's weights do not fit them (a second row tile
  // of an expert finds them in the XCD's L2).  MI355X, us, first / second product: 8 tokens top-2 of 64 experts 2048 x 8192
  // 91 / 86 -> 83 / 76 (5.6 and 6.2 TB/s); 96 tokens top-2 of 8 SwiGLU experts 4096 x 14336 338 / 180 -> 297 / 162 (6.3 and 5.8).
  // (past the last stage the descriptors are empty: nothing is read, and the number of loads in flight is always the same)
  auto issue_w = [&](auto policy, int kt, unsigned char* stage) __attribute__((always_inline)) {
    const bool live = kt < KT;
    const __amdgpu_buffer_rsrc_t rw = stream_rsrc(wa + wbase, live ? w_bytes : 0u);
#pragma unroll
    for (int i = 0; i < W_LOADS; ++i) {
      const int blk = block(i);
      __amdgpu_buffer_rsrc_t r = rw;
      if (EPI == ST_SWIGLU) r = stream_rsrc(((blk & 1) ? wb : wa) + wbase, live ? w_bytes : 0u);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)(stage + blk * 1024), 16, voff[i], kt * 128, 0,
                                               decltype(policy)::value);
    }
  };
  auto issue_a = [&](int kt, unsigned char* stage) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t ra = stream_rsrc(a_ptr, kt < KT ? a_bytes : 0u);
#pragma unroll
    for (int i = W_LOADS; i < LOADS; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (__attribute__((address_space(3))) void*)(stage + block(i) * 1024), 16, voff[i], kt * 128, 0, 0);
  };
  // ---- fragments: 16 rows x 32 values, lane = row + 16 * (chunk of the four)
  const int frow = lane & 15, fch = lane >> 4;
  const int wf = wave % S::NWF, wm = wave / S::NWF;  // row block b of row group wm is block b * NWM + wm of the tile
  const int in_row = frow * 128 + ((fch ^ ((frow >> 1) & 7)) << 4);   // (the key repeats every 16 rows) second 32 values: ^ 64
  const int w_off = wf * FB * 2048 + in_row, a_off = wm * 2048 + in_row;
  f32x4 acc[FB][RB];
#pragma unroll
  for (int f = 0; f < FB; ++f)
#pragma unroll
    for (int b = 0; b < RB; ++b) acc[f][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const unsigned char* ws, const unsigned char* as) __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      bf16x8 w[FB];
#pragma unroll
      for (int f = 0; f < FB; ++f) w[f] = *reinterpret_cast<const bf16x8*>(ws + (w_off ^ (kk << 6)) + f * 2048);
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        const bf16x8 r = *reinterpret_cast<const bf16x8*>(as + (a_off ^ (kk << 6)) + b * S::NWM * 2048);
#pragma unroll
        for (int f = 0; f < FB; ++f) acc[f][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[f], r, acc[f][b], 0, 0, 0);
      }
    }
    if constexpr (SPLIT) {
      // the next stages' loads between the multiplications: in one burst ahead of them the wavefronts wait for the queue
      __builtin_amdgcn_sched_group_barrier(0x100, FB + 1, 0);                         // DS read
#pragma unroll
      for (int q = 0; q < 2 * RB; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, FB, 0);                           // MFMA
        if (q + 2 == RB) __builtin_amdgcn_sched_group_barrier(0x100, FB + 1, 0);
        else __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        if (q < LOADS) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);             // VMEM
      }
    }
  };
  auto w_of = [&](auto i) -> unsigned char* {
    constexpr int I = decltype(i)::value % STAGES;
    if constexpr (I == 0) return w0;
    else if constexpr (I == 1) return w1;
    else if constexpr (I == 2) return w2;
    else if constexpr (I == 3) return w3;
    else return w4;
  };
  auto a_of = [&](auto i) -> unsigned char* {
    constexpr int I = decltype(i)::value % ROW_STAGES;
    if constexpr (I == 0) return a0;
    else if constexpr (I == 1) return a1;
    else if constexpr (I == 2) return a2;
    else if constexpr (I == 3) return a3;
    else return a4;
  };
  // Stage kt is multiplied while the weights of stages kt+1 .. kt+STAGES-1 (and the rows of kt+1 .. kt+ROW_STAGES-1) are on
  // their way.  A wavefront waits for its own share of stage kt (loads retire in order; a step requests rows before
  // weights) and for its reads of the stage before, then the workgroup meets: stage kt is whole and the buffers of stage
  // kt-1 are free.
  constexpr int AHEAD = ROW_STAGES == STAGES ? (STAGES - 2) * LOADS : (ROW_STAGES - 2) * LOADS + W_LOADS;
  auto step = [&](auto policy, auto i, int kt) __attribute__((always_inline)) {
    constexpr int I = decltype(i)::value;
    __builtin_amdgcn_s_waitcnt(wait_vm(AHEAD));
    __builtin_amdgcn_s_barrier();
    issue_a(kt + ROW_STAGES - 1, a_of(std::integral_constant<int, I + ROW_STAGES - 1>{}));
    if constexpr (SPLIT) __builtin_amdgcn_sched_barrier(0x0301);  // no load crosses: AHEAD counts on the weights being the younger ones
    issue_w(policy, kt + STAGES - 1, w_of(std::integral_constant<int, I + STAGES - 1>{}));
    compute(w_of(i), a_of(i));
  };
  constexpr int CYCLE = ROW_STAGES == STAGES ? STAGES : STAGES * ROW_STAGES, PASS = 24 / CYCLE * CYCLE;  // (3 and 2 stages: 6 steps)
  auto contract = [&](auto policy) {
    if constexpr (ROW_STAGES == STAGES) issue_a(0, a0);
    issue_w(policy, 0, w0);
    if constexpr (ROW_STAGES == STAGES) issue_a(1, a1);
    else issue_a(0, a0);
    issue_w(policy, 1, w1);
    if constexpr (STAGES > 3) { issue_a(2, a2); issue_w(policy, 2, w2); }
    if constexpr (STAGES > 4) { issue_a(3, a3); issue_w(policy, 3, w3); }
    if constexpr (OWN_TABLE) fill_phi_table(reinterpret_cast<phi_f32x2*>(table));  // (the steps' barriers are between it and its readers)
    // On every way round the loop all stages were requested, and inside a pass the compiler adds no wait of its own.  At the head
    // of the loop, where the passes and the prologue meet, it does: the first step of every pass waits for all loads (vmcnt(0)
    // behind the barrier), whichever stages they belong to.  So a pass is as many steps as come to about 24.
    // MI355X, whole layers against passes of three to six steps (us): 32 SwiGLU experts 4096 x 2048, 1500 tokens 396 / 373; 8 of
    // 2176 x 2048, 138 tokens, k 4 75.7 / 71.0; 64 of 2048 x 8192, 8 tokens 173 / 170, 4096 tokens: the second product 440 / 427.
    int kt = 0;
    auto pass = [&](auto... i) __attribute__((always_inline)) { return ((step(policy, i, kt), ++kt < KT) && ...); };
    while (unrolled<PASS>(pass)) {}
  };
  if (NT && t.tiles == 1) contract(std::integral_constant<int, LOAD_NT>{});
  else contract(std::integral_constant<int, 0>{});
  __builtin_amdgcn_s_waitcnt(wait_vm(0));  // (the empty loads retire)

  phi_f32x2* const phi = reinterpret_cast<phi_f32x2*>(OWN_TABLE ? table : w0);
  const float phi_add = phi_addend(phi);
  if constexpr (TABLE && !OWN_TABLE) {
    __syncthreads();
    fill_phi_table(phi);
    __syncthreads();
  }

  // ---- epilogue: lane holds weight rows 4 fch + 0..3 of every 16-row weight block, for row frow of every row block
#pragma unroll
  for (int f = 0; f < FB; ++f) {
    const int fblk = wf * FB + f;
    if (n0 + fblk * (EPI == ST_SWIGLU ? 8 : 16) < t.nt * OUTF) continue;  // (uniform; N is a multiple of 64)
    const int n = n0 + (EPI == ST_SWIGLU ? fblk * 8 + (fch & 1) * 4 : fblk * 16 + fch * 4);
    float bv[4] = {0.f, 0.f, 0.f, 0.f};
    if (EPI != ST_SWIGLU && bias) {
      const u32x2 b = *reinterpret_cast<const u32x2*>(bias + (eoff ? eoff[t.expert] : (int64_t)t.expert * N) + n);
      bv[0] = lo16(b.x); bv[1] = hi16(b.x); bv[2] = lo16(b.y); bv[3] = hi16(b.y);
    }
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      const int r = (b * S::NWM + wm) * 16 + frow;
      float p[4];
      if constexpr (EPI == ST_SWIGLU) {
        // the lower half of the lanes holds gate rows, lane + 32 the up rows of the same features and row: both get both
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t v = __float_as_uint(acc[f][b][i]);
          const u32x2 gu = __builtin_amdgcn_permlane32_swap(v, v, false, false);
          const float g = __uint_as_float(gu.x);
          p[i] = g * __builtin_amdgcn_rcpf(1.f + __expf(-g)) * __uint_as_float(gu.y);
        }
        if (lane >= 32) continue;
      }
      if (r >= t.rows) continue;
      size_t o = (size_t)(t.row0 + r) * N + n;
      if constexpr (EPI != ST_SWIGLU) {
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = acc[f][b][i] + bv[i];
      }
      if constexpr (TABLE) {
        gelu_table_n<4>(p, phi_add, phi);
      } else if constexpr (EPI == ST_GELU) {
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = gelu_exact(p[i]);
      }
      if constexpr (EPI == ST_COMBINE) {  // k = 1: the row's token
        const int token = row_map[t.row0 + r];
        o = (size_t)token * N + n;
        u32x2 res = {0u, 0u};
        if (residual) res = *reinterpret_cast<const u32x2*>(residual + o);
        const float g = gate_w[token];
        p[0] = fmaf(g, p[0], lo16(res.x)); p[1] = fmaf(g, p[1], hi16(res.x));
        p[2] = fmaf(g, p[2], lo16(res.y)); p[3] = fmaf(g, p[3], hi16(res.y));
      }
      *reinterpret_cast<u32x2*>(out + o) = u32x2{pack2(p[0], p[1]), pack2(p[2], p[3])};
    }
  }
#endif
}

template <int EPI, bool GATHER, typename S>
int32_t launch_shape(const moe_config* cfg, const uint16_t* act, const uint16_t* wa, const uint16_t* wb, const uint16_t* bias,
                     const int32_t* offsets, uint16_t* out, const int32_t* row_map, const float* gate_w, const uint16_t* residual,
                     const int32_t* a2r, const int64_t* eoff, int32_t* clear_ctr, int N, int K, hipStream_t s) {
  constexpr int OUTF = EPI == ST_SWIGLU ? S::WROWS / 2 : S::WROWS;
  const int n_tiles = (N + OUTF - 1) / OUTF;
  const int64_t grid = row_tile_grid(cfg, S::TM, n_tiles);
  if (grid > INT32_MAX) return fail(MOE_ERR_UNSUPPORTED, "expert stream: too many tiles");
  if (max_rows(cfg) == 0) return MOE_OK;
  auto kern = weights_exceed_cache(cfg) ? expert_stream_kernel<EPI, GATHER, true, S> : expert_stream_kernel<EPI, GATHER, false, S>;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(S::WAVES * 64), 0, s, act, wa, wb, bias,
                     offsets, out, row_map, gate_w, residual, a2r, eoff, clear_ctr, cfg->T, cfg->E, N, K, n_tiles);
  return check_hip(hipGetLastError(), "expert stream launch");
}

// Which shape (weight rows x rows) serves a product of N features over K values, for evenly loaded experts (every shape
// handles any routing); none: the grouped GEMM.  Measured on MI355X (us, grouped GEMM / here), rows = rows per expert:
//  - up to 24 rows the time is the weights': 64x32, three workgroups per CU.  SwiGLU d 4096, f 14336, 8 experts, 24 rows:
//    386 / 359 and, with 128 big tiles for 256 CUs, 329 / 165;
//  - up to 44 rows 256x64 and up to 96 rows 256x128 where such tiles come in nearly whole rounds of the chip (one workgroup
//    per CU, twice the weights per stage).  64 experts, d 2048, f 8192, 32 rows: 396 / 363 and 386 / 366 (128x64: 378 and
//    363); 64 rows 439 / 394 and 430 / 368; 94 rows 445 / 409 and 428 / 379; 128 SwiGLU experts, 1600 x 832, 38 rows 175 / 145;
//  - up to 36 otherwise: 128x64.  64 experts, 1280 x 1280, 30 rows 47 / 37;
//  - few tiles of any kind: 64x64.  4 experts, 150 rows, d 320, f 1088: 9.2 / 2.0 and 18.8 / 5.2;
//  - up to 96 rows with long rows of weights or few big tiles: 128x128.  8 experts of 4096 x 14336, 40 rows 230 / 204; 32
//    experts, f 2560 -> d 1664, 62 rows 66 / 58; but f 8192 -> d 2048, 64 experts, 107 rows (some over 128) 428 / 474;
//  - few big tiles: 128x192 as long as they are one round, or two with long rows.  16 experts, f 4096 -> d 1024, 256 rows
//    (64 big tiles) 86 / 49; 8 experts, f 3072 -> d 768, 750 rows (72) 59 / 33; 8 experts, f 14336 -> d 4096 (128), 128 rows
//    347 / 203, 175 rows with uneven routing 355 / 367; two rounds of short rows: 16 experts, f 704 -> d 1408, 209 rows 22.7 / 23.4;
//  - three quarters of a round of big tiles against at most two rounds of 128x128 (with a whole round of them the big tiles
//    win: 16 experts, d 1024 -> f 4096, 128 rows 29 / 31, uneven 28 / 46).  16 experts, f 8704 -> d 640, 590 rows (144) 194 /
//    171 and, with Zipf(1.2) routing, 238 / 169; f 1408 -> d 1216, 330 rows 31 / 28, but 381 rows, where an uneven routing takes
//    a fourth row tile, 33 / 39.  97 to 192 rows gain at most a tenth and lose a fifth to the same edge;
//  - beyond one round, short rows: these workgroups are not persistent, so every tile pays its own start and end (a SwiGLU
//    tile has two products to spread them over).  Over 4400 random shapes and 600 of 448 to 1300 values, even routing, grouped
//    / here: 128x64 (where 256x64 does not serve), SwiGLU up to 576 values 0.96 (0.88 at worst), above 1.0 to 1.3; others up to
//    768 0.9 (0.74), from 832 1.0 to 1.1 where the big tiles leave a fifth of their rounds empty, where they do not 0.86 to
//    1.07 up to 1024 and 1.05 and more above; 256x128 up to 704 0.97 to 1.02 (0.86), above 1.04 to 1.14; 128x128 below 2048 1.02
//    (0.90).
//  - 37 to 96 rows otherwise: 256x128 instead of the grouped GEMM, by what the tile's end costs.  Layers under even / Zipf(1.2)
//    routing, in brackets how many are more than 2 % slower: SwiGLU from 768 values 1.130 over 841 (0) / 1.135 over 553 (43); plain from
//    512 1.077 over 1518 (4) / 1.096 over 945 (41); combine, whose end waits for row numbers, gate weights and residual rows, from
//    832 1.075 over 439 (2) / 1.092 over 266 (18), but 512 to 831 1.012 over 290 (30) / 1.004 over 214 (63; 64 experts 640 -> 832, 77
//    rows, even 96 / 107).  Up to a quarter below its line each has 1.02 to 1.06 and 2 to 4 % of its layers slower, under Zipf up to 18 %.
//    GELU ends do not wait longer than plain ones: from 640 values on 1.108 over 1001 (1) / 1.126 over 519 (30).  The rule takes fewer,
//    1.113 over 512 (1) / 1.136 over 314 (18): below 1088 values only where the last round is nearly full; the rest (489 products 1.10,
//    none slower) stays on the lines of the time when the table was built behind the K loop.
//  - up to 96 rows, long rows of weights: one round of 256x128 where 128x128 makes more than one (128x128 / 256x128): even routing
//    1.075 over 377 (0), Zipf(1.2) 1.037 over 329 (29).  Where 128x128 is one round too, 0.90 over 3332 (12 SwiGLU experts 3584 -> 1344, 83
//    rows, 132 tiles against 252: 92 / 110).  Under Zipf a hot expert's further row tiles open a second round: of the products of any
//    width 129 to 176 tiles 1.05 over 488 (27), more of up to 12 experts 1.03 over 168 (44), more of 16 to 96 experts 1.00 over 728 (256;
//    24 experts 4608 -> 1088, 55 rows, 216 tiles: 202 / 239), though 1.06 under even routing.  Narrower products with an activation
//    and lengths beyond 4608 gain as much (1.080 over 384 (0) / 1.036 over 270 (24)) and stay on 128x128 all the same: the rule keeps
//    to what it had.
//  - 97 to 160 rows otherwise: 256x192, three stages of weights and two of rows in the LDS; the grouped GEMM has one stage of
//    weights on its way and waits for it.  Over 126 random products of 97 to 180 rows 1.12 on average (grouped / here): 64
//    experts, 131 rows, f 3456 -> d 3264 366 / 314; 16 SwiGLU, 112 rows, 3008 -> 8704 467 / 398; 64 SwiGLU, 128 rows, 2048 -> 4096
//    523 / 466 and 283 / 210; few tiles 1.2 to 1.3.  Layers under even / Zipf(1.2) routing, as above: GELU 1.071 over 493 (5) / 1.062
//    over 216 (20), SwiGLU 1.072 over 749 (3) / 1.092 over 396 (39), plain 1.060 over 833 (9) / 1.072 over 381 (31), combine 1.068 over
//    129 (4) / 1.096 over 52 (4).  Not beyond 160 rows, where experts need a second tile (32 experts, 169 rows, 5248 -> 3904 326 /
//    350).  Not for rows of weights below 704 values, where the start and end of these tiles weigh: 512 to 703 SwiGLU 1.013 over 306 (60) /
//    0.975, plain 1.031 over 143 (3) / 1.009 over 77 (15), GELU 1.041 over 287 (5) / 0.992 over 52 (21).  More than six rounds
//    with an activation: from 2240 on, as the grouped GEMM's persistent workgroups hide ends (SwiGLU 704 to 2239 0.987 over 52).
//    Combines from 2560 on (1152 to 2559 1.020 over 173 (7) / 1.014 over 66 (16); 32 experts, 134 rows, 1984 -> 4032 142 / 156).  GELU products
//    of at most 192 tiles stay with the grouped GEMM on an older line; they would gain 1.07 (204 from 704 values on, none slower).
//    Nor where an expert is likely to need a second tile (from 135 rows on: random routing spreads rows by a tenth to an eighth) and
//    the tiles leave no room for it in their last round (64 experts, 142 rows, 2752 -> 896 94 / 128).
//  Whole layers above: 20900 random ones of 25 to 176 rows, both products on every shape in turn, two to four sets of weights in turn.
// Skewed routing costs row tiles that the rule does not see.  Over the same shapes under Zipf(1.2) masses the mean gain is
// within a tenth of that under even routing, but 128x192 loses 7 to 14 % where the hot expert's extra tiles open a second
// round (16 experts, f 1600 -> d 1792, 115 rows: even 33 / 22, Zipf 35 / 40), and 64x32 up to 20 % with every row of a
// step on one expert of 64.  Of 1300 whole expert blocks under even or random routing none was more than 3 % slower than on
// the grouped GEMM, of 1300 under Zipf or half-on-one-expert routing 16 were, by up to 9 % (before the shapes of 256 weight rows;
// theirs stand with them).
enum { STREAM_NONE, STREAM_64x32, STREAM_64x64, STREAM_128x64, STREAM_128x128, STREAM_128x192, STREAM_256x64, STREAM_256x128, STREAM_256x192 };
int pick_stream(const moe_config* cfg, int N, int K, int epi) {
  const bool swiglu = epi == ST_SWIGLU, activation = epi == ST_GELU || swiglu;
  if (cfg->dtype != MOE_BF16 || N % 64 || K % ST_KS) return STREAM_NONE;
  // Buffer sizes and offsets of a tile are 32-bit.  The line is that of the grouped GEMM's largest row tile, so that what
  // that kernel refuses stays refused whichever of the two would serve the row count.
  if ((int64_t)320 * K * 2 >= ((int64_t)1 << 31)) return STREAM_NONE;
  // (the switches ask for the grouped GEMM's kernels)
  if (!tuning(MOE_TUNE_FEW_TOKEN_KERNELS) || tuning(MOE_TUNE_GEMM_TILE_ROWS) || tuning(MOE_TUNE_GEMM_MFMA)) return STREAM_NONE;
  int64_t rows = ((int64_t)cfg->k * cfg->T + cfg->E - 1) / cfg->E;
  const int64_t C = moe_capacity(cfg);
  if (rows > C) rows = C;
  if (rows <= 24) return STREAM_64x32;
  // tiles of fr weight rows x tm rows, for `each` rows per expert
  auto tiles_of = [&](int fr, int tm, int64_t each) {
    const int outf = swiglu ? fr / 2 : fr;
    return cfg->E * ((each + tm - 1) / tm) * ((N + outf - 1) / outf);
  };
  auto tiles = [&](int fr, int tm) { return tiles_of(fr, tm, rows); };
  auto one_round = [&](int fr, int tm) { return tiles(fr, tm) <= 256; };
  const int64_t big = tiles(256, 256);
  const bool wide = N >= (swiglu ? 64 : 128);
  // share of its rounds of 256 workgroups (one per CU) that a shape of 256 weight rows fills
  auto fill = [&](int tm) {
    const int64_t t = N >= (swiglu ? 128 : 256) ? tiles(256, tm) : 0;
    return t < 256 ? 0.0 : (double)t / (double)((t + 255) / 256 * 256);
  };
  if (rows <= 44 && fill(64) >= 0.95 && (one_round(256, 64) || K >= 768)) return STREAM_256x64;
  const bool big_fit = 5 * big >= 4 * ((big + 255) / 256 * 256);  // the big tiles fill four fifths of their rounds
  if (wide && rows <= 36 && (one_round(128, 64) || K >= (swiglu ? 640 : big_fit ? 1088 : 832))) return STREAM_128x64;
  if (tiles(128, 192) < 128 && tiles(64, 64) <= 512) return STREAM_64x64;
  const bool long_rows = K >= 4096 || big < 256;
  if (rows <= 96 && fill(128) >= (long_rows ? 0.95 : 0.85) && (one_round(256, 128) || K >= (swiglu ? 768 : 832))) return STREAM_256x128;
  // (one round of the wider tiles where 128 weight rows make more than one; more experts: with room for a hot one's further row tiles)
  const bool one_of_256 = N >= (swiglu ? 768 : epi == ST_GELU ? 2048 : 256) && K <= 4608 && !one_round(128, 128) &&
                          tiles(256, 128) <= (cfg->E < 16 ? 256 : 176);
  if (wide && rows <= 96 && long_rows && (one_round(128, 128) || K >= 2048)) return one_of_256 ? STREAM_256x128 : STREAM_128x128;
  if (wide && (big <= 96 || (big <= 128 && rows <= 152)) && tiles(128, 192) <= (K >= 4096 ? 512 : 256)) return STREAM_128x192;
  // (8 % head-room for uneven routing, like the grouped GEMM's choice: a row tile more would be a round more)
  if (wide && rows > 192 && big > 128 && big <= 192 && tiles_of(128, 128, rows + (rows * 2 + 24) / 25) <= 512) return STREAM_128x128;
  if (N < (swiglu ? 128 : 256)) return STREAM_NONE;
  const int shortest = swiglu ? 768 : epi == ST_COMBINE ? 832 : 512;
  if (rows <= 96 && (epi == ST_GELU ? K >= 1088 || (K >= 640 && fill(128) >= 0.83) : K >= shortest)) return STREAM_256x128;
  if (rows > 96 && rows <= 160) {
    const int64_t t = tiles(256, 192), rounds = (t + 255) / 256;
    if (rows > 134 && C > 192 && 100 * t > 97 * 256 * rounds) return STREAM_NONE;
    if (epi == ST_COMBINE) return K >= 2560 ? STREAM_256x192 : STREAM_NONE;
    if (K >= (activation && t > 6 * 256 ? 2240 : 704) && !(epi == ST_GELU && t <= 192)) return STREAM_256x192;
  }
  return STREAM_NONE;
}

template <int EPI, bool GATHER>
int32_t launch(const moe_config* cfg, const uint16_t* act, const uint16_t* wa, const uint16_t* wb, const uint16_t* bias,
               const int32_t* offsets, uint16_t* out, const int32_t* row_map, const float* gate_w, const uint16_t* residual,
               const int32_t* a2r, const int64_t* eoff, int32_t* clear_ctr, int N, int K, hipStream_t s) {
#define MOE_STREAM(...) return launch_shape<EPI, GATHER, StreamShape<__VA_ARGS__>>(cfg, act, wa, wb, bias, offsets, out, row_map, gate_w, residual, a2r, eoff, clear_ctr, N, K, s)
  switch (pick_stream(cfg, N, K, EPI)) {
    case STREAM_64x32: MOE_STREAM(4, 1, 1, 2, 4);
    case STREAM_64x64: MOE_STREAM(4, 1, 1, 4, 4);
    case STREAM_128x64: MOE_STREAM(4, 2, 2, 2, 5);
    case STREAM_128x128: MOE_STREAM(4, 2, 2, 4, 4);
    case STREAM_128x192: MOE_STREAM(4, 2, 2, 6, 4);
    case STREAM_256x64: MOE_STREAM(4, 2, 4, 2, 4);
    case STREAM_256x128: MOE_STREAM(4, 2, 4, 4, 3);
    case STREAM_256x192: MOE_STREAM(4, 2, 4, 6, 3, 2);
  }
#undef MOE_STREAM
  return fail(MOE_ERR_UNSUPPORTED, "expert stream: shape outside its range");
}

}  // namespace

bool expert_stream_applies(const moe_config* cfg, int N, int K, int epi) { return pick_stream(cfg, N, K, epi) != STREAM_NONE; }

// name of the shape (weight rows x rows), for tests
const char* expert_stream_shape(const moe_config* cfg, int N, int K, int epi) {
  static const char* const names[] = {"", "stream 64x32", "stream 64x64", "stream 128x64", "stream 128x128", "stream 128x192", "stream 256x64", "stream 256x128", "stream 256x192"};
  return names[pick_stream(cfg, N, K, epi)];
}

// epi: 0 GELU (+bias), 1 SwiGLU (wa = gate, wb = up), 2 plain (+bias), 3 combine for k = 1 (row_map = row_to_assign,
// gate_w, residual; a2r or NULL: fill_rowless_tokens).  row_map with epi 0/1: gather the rows from x[T, K].  eoff: per-expert element offsets or NULL.
// clear_ctr (nullable): eight ints cleared on the way, the tile counters that the grouped GEMM in this place would clear.
int32_t launch_expert_stream_bf16(int epi, const moe_config* cfg, const void* act, const void* wa, const void* wb, const void* bias,
                                  const int32_t* offsets, void* out, const int32_t* row_map, const float* gate_w,
                                  const void* residual, const int32_t* a2r, const int64_t* eoff, int32_t* clear_ctr, int N, int K, hipStream_t s) {
  const uint16_t *a = (const uint16_t*)act, *w0 = (const uint16_t*)wa, *w1 = (const uint16_t*)wb, *b = (const uint16_t*)bias;
  const uint16_t* res = (const uint16_t*)residual;
  uint16_t* o = (uint16_t*)out;
  switch (epi) {
    case ST_GELU:
      return row_map ? launch<ST_GELU, true>(cfg, a, w0, w1, b, offsets, o, row_map, gate_w, res, a2r, eoff, clear_ctr, N, K, s)
                     : launch<ST_GELU, false>(cfg, a, w0, w1, b, offsets, o, row_map, gate_w, res, a2r, eoff, clear_ctr, N, K, s);
    case ST_SWIGLU:
      return row_map ? launch<ST_SWIGLU, true>(cfg, a, w0, w1, nullptr, offsets, o, row_map, gate_w, res, a2r, eoff, clear_ctr, N, K, s)
                     : launch<ST_SWIGLU, false>(cfg, a, w0, w1, nullptr, offsets, o, row_map, gate_w, res, a2r, eoff, clear_ctr, N, K, s);
    case ST_BIAS: return launch<ST_BIAS, false>(cfg, a, w0, w1, b, offsets, o, nullptr, gate_w, res, a2r, eoff, clear_ctr, N, K, s);
    case ST_COMBINE:
      if (!row_map || !gate_w || cfg->k != 1) return fail(MOE_ERR_INVALID_ARG, "expert stream: combine epilogue needs k = 1, row map and gate weights");
      return launch<ST_COMBINE, false>(cfg, a, w0, w1, b, offsets, o, row_map, gate_w, res, a2r, eoff, clear_ctr, N, K, s);
  }
  return fail(MOE_ERR_INVALID_ARG, "expert stream: unknown epilogue");
}

}  // namespace moesys
