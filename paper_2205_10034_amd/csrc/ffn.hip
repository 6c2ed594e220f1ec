// Expert FFN entry point, the float32 grouped GEMM (correctness configuration)
// and the one-time expert weight transpose.
//
// The bf16 MFMA grouped GEMM lives in grouped_gemm_bf16.hip; the float32 path
// below multiplies on the float32 matrix instructions.
#include <cmath>
#include <type_traits>
#include "moesys_internal.h"
#include "row_tiles.h"
#include "wave_util.h"

namespace moesys {

int32_t launch_gemm1_bf16(const moe_config*, const moe_weights*, const void*, const int32_t*, void*, const int32_t*, int32_t*,
                          hipStream_t);
int32_t launch_gemm2_bf16(const moe_config*, const moe_weights*, const void*, const int32_t*, void*, int32_t*, hipStream_t);
int32_t launch_gemm2_combine_bf16(const moe_config*, const moe_weights*, const void*, const int32_t*, const int32_t*,
                                  const float*, const void*, void*, const int32_t*, int32_t*, hipStream_t);

namespace {

enum { F_GELU = 0, F_SWIGLU = 1, F_BIAS = 2 };

__device__ __forceinline__ float gelu_exact(float u) { return 0.5f * u * (1.f + erff(u * 0.70710678118654752f)); }
__device__ __forceinline__ float silu_exact(float u) { return u / (1.f + expf(-u)); }

// Four floats from any float address (one 16-byte load; the hardware asks for no more than 4-byte alignment).
typedef float f32x4a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
__device__ __forceinline__ f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4a4*>(p); }

// What a layer's products take over from the kernels around them, a launch of 3 to 6 us each.  First product: act is x and row r
// reads token row_map[r] mod T; the tiles of a row's features store their share of the dispatched rows in xd.  Second
// product, k = 1: it writes out[token] = residual[token] + gate_w[token] * row as well; rowless tokens (a2r < 0) get their residual
// or zero from the workgroups together.  NULL pointers: not asked for.  Measured on MI355X, whole layers (us, before / now): 256
// tokens 128 x 512 of 4 experts, k 1 27.3 / 20.8; 996, 960 x 832, 4, k 1 76.9 / 69.2; 381, 960 x 1408, 16, k 2 112 / 102; 2048, 1024 x
// 4096, 16, k 2 710 / 705.
struct F32Layer {
  const int32_t* row_map;
  float* xd;
  const float* gate_w;
  const float* residual;
  float* out;
  const int32_t* a2r;
  int T;
};
__device__ __forceinline__ int act_row(const F32Layer& l, int row) {
  if (!l.xd) return row;
  int t = l.row_map[row];
  while (t >= l.T) t -= l.T;  // assignment id j*T + t -> token (j < k <= 8)
  return t;
}
// A tile's share of the dispatched rows: rows nt, nt + n_tiles, ... of its row tile, in 16-byte pieces.  The first piece of a thread
// is requested before the product and stored after it.
struct RowShare { size_t at; f32x4 v; };
__device__ __forceinline__ RowShare share_piece(const F32Layer& l, const float* x, const RowTile& t, int n_tiles, int K, int i) {
  const int q = i / (K / 4), r = t.nt + q * n_tiles, c = 4 * (i - q * (K / 4));
  RowShare p = {~(size_t)0, f32x4{0.f, 0.f, 0.f, 0.f}};
  if (r < t.rows) {
    p.at = (size_t)(t.row0 + r) * K + c;
    p.v = load4(x + (size_t)act_row(l, t.row0 + r) * K + c);
  }
  return p;
}
__device__ __forceinline__ RowShare first_share(const F32Layer& l, const float* x, const RowTile& t, int n_tiles, int K) {
  return l.xd ? share_piece(l, x, t, n_tiles, K, threadIdx.x) : RowShare{~(size_t)0, f32x4{0.f, 0.f, 0.f, 0.f}};
}
__device__ __forceinline__ void combine_one(const F32Layer& l, int row, int N, int n, float y) {
  const int token = l.row_map[row];  // (k = 1: the assignment is the token)
  const size_t o = (size_t)token * N + n;
  l.out[o] = fmaf(l.gate_w[token], y, l.residual ? l.residual[o] : 0.f);
}
template <int THREADS>
__device__ __forceinline__ void store_share(const F32Layer& l, const float* x, const RowTile& t, int n_tiles, int K, RowShare p) {
  if (!l.xd) return;
  for (int i = threadIdx.x; p.at != ~(size_t)0; p = share_piece(l, x, t, n_tiles, K, i += THREADS)) *reinterpret_cast<f32x4a4*>(l.xd + p.at) = p.v;
}

// out[r, n] = epi(sum_k act[r,k] * W_e(n,k) (+ bias)) in float32 on v_mfma_f32_32x32x2_f32 (fused multiply-adds, float32
// accumulation): out rows are the MFMA's rows, output features its columns.  Lane l supplies row (column) l mod 32 and,
// of eight consecutive values of the contraction index, the four of its half l / 32: the order of a dot product's terms
// is free, so four MFMAs of two values each take one 16-byte piece per lane and operand.
// OUTPUT_MAJOR weights [n][k] are such pieces already; INPUT_MAJOR ones [k][n] (IM) are read one value per lane, 32
// consecutive features at a time.
// Many tiles: 64 rows x 64 features per workgroup, four wavefronts of 32 x 32, 32 values of the contraction index per
// step.  A step's operands go through registers into one of two LDS stages while the other is multiplied (rows padded
// to 36 floats: the 16-byte reads of 16 rows hit all banks once); one barrier per step.  Bound by the float32 MFMA rate
// (1024 clocks per step) once several workgroups per CU cover each other's barriers; small tiles, because an expert's last
// row tile is half empty on average and experts are many.  (64 x 128 tiles measured 2-30 % slower except for INPUT_MAJOR
// weights at the largest size, 346 against 353 us.)  SwiGLU: a gate block and the up block of the same features per wavefront.
// Measured on MI355X at 4096 rows over 16 experts, d_model 1024, d_ff 4096 (two products of 34.4 GFLOP): 764 + 837 us on
// the vector ALU (10 times that without a capacity bound: its grid had a workgroup for every row tile of every expert),
// 350 + 371 us here (98 and 93 TFLOP/s of the 154 that the vendor's dense product of 8192^3 reaches).
constexpr int FM = 64, FN = 64, FKS = 32, FPITCH = FKS + 4;  // rows and output features per tile, values per step, LDS pitch
template <int EPI, bool IM>
__global__ __launch_bounds__(256, 2) void ffn_f32_kernel(const float* __restrict__ act, const float* __restrict__ wa,
                                                         const float* __restrict__ wb, const float* __restrict__ bias,
                                                         const int32_t* __restrict__ offsets, float* __restrict__ out, int E,
                                                         int N, int K, int n_tiles, F32Layer layer) {
  constexpr int NB = EPI == F_SWIGLU ? 2 : 1;          // 32-feature blocks per wavefront
  constexpr int TN = FN * NB;                          // weight rows per tile
  constexpr int BP = IM ? TN + 4 : FPITCH, BROWS = IM ? FKS : TN;
  __shared__ __attribute__((aligned(16))) float sa[2][FM * FPITCH];
  __shared__ __attribute__((aligned(16))) float sb[2][BROWS * BP];
  RowTile t;
  if (EPI == F_BIAS && layer.out) fill_rowless_tokens<4>(layer.a2r, offsets[E], layer.T, N, layer.residual, layer.out);
  if (!find_row_tile<FM>(offsets, E, n_tiles, t)) return;
  const RowShare share = first_share(layer, act, t, n_tiles, K);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wc = wave >> 1, l32 = lane & 31, h = lane >> 5;
  const int n0 = t.nt * FN;
  const size_t we = (size_t)t.expert * N * K;

  // this thread's 16-byte pieces of a stage: two of the rows, TN / 32 of the weights; pieces past the last row or
  // feature re-read the last one
  const float* pa[2];
  const float* pb[TN / 32];
  int la[2], lb[TN / 32];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int i = q * 256 + tid, r = i / 8, c = i % 8;
    pa[q] = act + (size_t)act_row(layer, t.row0 + min(r, t.rows - 1)) * K + 4 * c;
    la[q] = r * FPITCH + 4 * c;
  }
#pragma unroll
  for (int q = 0; q < TN / 32; ++q) {
    const int i = q * 256 + tid;
    const int r = IM ? i / (TN / 4) : i / 8, c = IM ? i % (TN / 4) : i % 8;  // IM: contraction row r, features 4c; else feature r
    const int f = IM ? 4 * c : r;                                            // feature inside the tile
    const float* w = EPI == F_SWIGLU && f >= FN ? wb : wa;
    const int n = EPI == F_SWIGLU && f >= FN ? n0 + f - FN : n0 + f;
    if (IM) pb[q] = w + we + (size_t)r * N + min(n, N - 4);                   // (N is a multiple of 64)
    else pb[q] = w + we + (size_t)min(n, N - 1) * K + 4 * c;
    lb[q] = r * BP + 4 * c;
  }
  const size_t b_step = IM ? (size_t)FKS * N : FKS;
  f32x4 ra[2], rb[TN / 32];
  auto load = [&](int kt) {
#pragma unroll
    for (int q = 0; q < 2; ++q) ra[q] = load4(pa[q] + (size_t)kt * FKS);
#pragma unroll
    for (int q = 0; q < TN / 32; ++q) rb[q] = load4(pb[q] + kt * b_step);
  };
  auto store = [&](int s) {
#pragma unroll
    for (int q = 0; q < 2; ++q) *reinterpret_cast<f32x4*>(&sa[s][la[q]]) = ra[q];
#pragma unroll
    for (int q = 0; q < TN / 32; ++q) *reinterpret_cast<f32x4*>(&sb[s][lb[q]]) = rb[q];
  };
  f32x16 acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
  auto compute = [&](int s) {
#pragma unroll
    for (int kk = 0; kk < FKS / 8; ++kk) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(&sa[s][(wm * 32 + l32) * FPITCH + kk * 8 + 4 * h]);
      f32x4 b[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int f = j * FN + wc * 32 + l32;
        if (IM) {
#pragma unroll
          for (int i = 0; i < 4; ++i) b[j][i] = sb[s][(kk * 8 + 4 * h + i) * BP + f];
        } else {
          b[j] = *reinterpret_cast<const f32x4*>(&sb[s][f * BP + kk * 8 + 4 * h]);
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j][i], acc[j], 0, 0, 0);
    }
  };
  const int KT = K / FKS;  // K is a multiple of 64
  const bool busy = wm * 32 < t.rows;  // (a wavefront without a row leaves the matrix pipe to the others)
  load(0);
  store(0);
  load(1);
  __syncthreads();
  for (int kt = 0; kt < KT; ++kt) {
    if (kt + 1 < KT) store((kt + 1) & 1);       // (nobody has read that stage since the last barrier)
    if (kt + 2 < KT) load(kt + 2);
    if (busy) compute(kt & 1);
    __syncthreads();
  }
  // register v of lane (l32, h): row (v & 3) + 8 (v >> 2) + 4 h of the wavefront's 32, feature l32 of the block
  const int n = n0 + wc * 32 + l32;  // (N is a multiple of 64)
  const float b = EPI != F_SWIGLU && bias ? bias[(size_t)t.expert * N + n] : 0.f;
  // What a combine reads is requested together, ahead of the stores, which may be in the same place.  (8 experts 512 x 2048, 3000
  // tokens: 182 us a layer row by row, 176 together.  INPUT_MAJOR weights: the registers cost a workgroup per CU, 43.6 / 46.2.)
  constexpr bool TOGETHER = EPI == F_BIAS && !IM;
  size_t at[TOGETHER ? 16 : 1];
  float gw[TOGETHER ? 16 : 1], res[TOGETHER ? 16 : 1];
  if constexpr (TOGETHER) {
    if (layer.out) {
      int token[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) token[v] = layer.row_map[t.row0 + min(wm * 32 + (v & 3) + 8 * (v >> 2) + 4 * h, t.rows - 1)];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        at[v] = (size_t)token[v] * N + n;
        gw[v] = layer.gate_w[token[v]];
        res[v] = layer.residual ? layer.residual[at[v]] : 0.f;
      }
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int r = wm * 32 + (v & 3) + 8 * (v >> 2) + 4 * h;
    if (r >= t.rows) continue;
    float u = acc[0][v];
    if constexpr (EPI == F_SWIGLU) u = silu_exact(u) * acc[NB - 1][v];
    else if (EPI == F_GELU) u = gelu_exact(u + b);
    else u += b;
    out[(size_t)(t.row0 + r) * N + n] = u;
    if constexpr (TOGETHER) {
      if (layer.out) layer.out[at[v]] = fmaf(gw[v], u, res[v]);
    } else if (EPI == F_BIAS && layer.out) {
      combine_one(layer, t.row0 + r, N, n, u);
    }
  }
  store_share<256>(layer, act, t, n_tiles, K, share);
}

// Up to 16 BU rows x 64 FBW weight rows per workgroup, four wavefronts of 16 FBW weight rows each on v_mfma_f32_16x16x4_f32,
// weights as the first operand: a lane ends up with four consecutive features of one row.  An expert's rows are dealt out
// evenly over the fewest tiles in units of 16, and the K loop is compiled once per number of units, so a tile multiplies what
// it holds.  A step is 32 values of the contraction index: operands go through registers into one of two LDS stages (16-byte
// chunks XORed with half the row) while the other is multiplied; the loads of the step after next stay in flight across the
// barrier, and a unit's rows of the second half of a step are read as soon as those of the first have been multiplied.
// Two shapes, by pick_f32: 80 rows, three workgroups per CU (SwiGLU: 128 weight rows, two products; two per CU if input-major), and
// 160 rows x 128 weight rows, two per CU.  Bound by the float32 MFMAs (busy 75 % with even rows) and by whole rounds of tiles.  Measured on MI355X
// against the 64 x 64 kernel (us): 80 rows, 140 random products 1.07 on average where the rule below picks it, 1.10 each
// (4 experts of 1538 rows, 3712 -> 192 149 / 106; 8 of 268, 3648 -> 960 206 / 164; 16 of 69, 768 -> 3584 114 / 82); 160 rows, 16
// experts of 256, 1024 -> 4096 -> 1024: 354 / 322 and 375 / 334 (107 and 103 TFLOP/s).
template <int EPI, bool IM, int FBW, int BU>
__global__ __launch_bounds__(256, BU > 5 ? 2 : 3) void ffn_f32_units_kernel(const float* __restrict__ act, const float* __restrict__ wa,
                                                                          const float* __restrict__ wb, const float* __restrict__ bias,
                                                                          const int32_t* __restrict__ offsets, float* __restrict__ out,
                                                                          int E, int N, int K, int n_tiles, F32Layer layer) {
  constexpr int BM = 16 * BU;
  static_assert(EPI != F_SWIGLU || FBW == 2, "a wavefront has a gate block and the up block of the same features");
  constexpr int TN = 64 * FBW, OUTF = EPI == F_SWIGLU ? TN / 2 : TN;  // weight rows, output features
  constexpr int AQ = (BM * 8 + 255) / 256, BQ = TN * 8 / 256;                 // 16-byte pieces of a stage per thread
  constexpr int BP = TN + 4;                                          // IM: LDS pitch of a row of weights, in floats
  __shared__ __attribute__((aligned(16))) float sa[2][BM * FKS];
  __shared__ __attribute__((aligned(16))) float sb[2][IM ? FKS * BP : TN * FKS];
  RowTile t;
  if (EPI == F_BIAS && layer.out) fill_rowless_tokens<4>(layer.a2r, offsets[E], layer.T, N, layer.residual, layer.out);
  if (!find_row_tile<BM, 16>(offsets, E, n_tiles, t)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q16 = lane & 15, g = lane >> 4;
  const int n0 = min(t.nt * OUTF, N - OUTF);  // (the last tile of a feature count that is no multiple leaves to the one before what is its)
  const size_t we = (size_t)t.expert * N * K;
  const int units = (t.rows + 15) / 16;
  // weight row r of the tile: matrix and feature (SwiGLU: 16 gate rows and 16 up rows of the same features per wavefront)
  auto feature = [&](int r) { return EPI == F_SWIGLU ? n0 + (r >> 5) * 16 + (r & 15) : n0 + r; };
  auto matrix = [&](int r) { return EPI == F_SWIGLU && (r & 16) ? wb : wa; };

  const float* pa[AQ];
  const float* pb[BQ];
  int la[AQ], lb[BQ];
#pragma unroll
  for (int q = 0; q < AQ; ++q) {
    const int i = q * 256 + tid, r = i / 8, c = i % 8;
    pa[q] = act + (size_t)act_row(layer, t.row0 + min(r, t.rows - 1)) * K + 4 * c;
    la[q] = r * FKS + 4 * (c ^ ((r >> 1) & 7));
  }
#pragma unroll
  for (int q = 0; q < BQ; ++q) {
    const int i = q * 256 + tid;
    if (IM) {
      const int kr = i / (TN / 4), r = 4 * (i % (TN / 4));  // contraction row, first of four weight rows
      pb[q] = matrix(r) + we + (size_t)kr * N + feature(r);
      lb[q] = kr * BP + r;
    } else {
      const int r = i / 8, c = i % 8;
      pb[q] = matrix(r) + we + (size_t)feature(r) * K + 4 * c;
      lb[q] = r * FKS + 4 * (c ^ ((r >> 1) & 7));
    }
  }
  const size_t b_step = IM ? (size_t)FKS * N : FKS;
  const int w0 = wave * 16 * FBW, key = (q16 >> 1) & 7;  // (the key of a row repeats every 16)
  const int KT = K / FKS;
  f32x4 acc[BU][FBW];
#pragma unroll
  for (int u = 0; u < BU; ++u)
#pragma unroll
    for (int f = 0; f < FBW; ++f) acc[u][f] = f32x4{0.f, 0.f, 0.f, 0.f};
  // the K loop of a tile of U units: 16 values at a time, of which lane group g has the four of chunk 4 h + g, one per MFMA
  auto contract = [&](auto u_tag) {
    constexpr int U = decltype(u_tag)::value, AU = (U + 1) / 2;
    f32x4 ra[AU], rb[BQ], x[U], w[2][FBW];
    auto load = [&](int kt) {
#pragma unroll
      for (int q = 0; q < AU; ++q) ra[q] = load4(pa[q] + (size_t)kt * FKS);
#pragma unroll
      for (int q = 0; q < BQ; ++q) rb[q] = load4(pb[q] + kt * b_step);
    };
    auto store = [&](int s) {
#pragma unroll
      for (int q = 0; q < AU; ++q)
        if (32 * q + 32 <= BM || tid < (BM - 32 * q) * 8)  // (BM is a multiple of 16)
          *reinterpret_cast<f32x4*>(&sa[s][la[q]]) = ra[q];
#pragma unroll
      for (int q = 0; q < BQ; ++q) *reinterpret_cast<f32x4*>(&sb[s][lb[q]]) = rb[q];
    };
    auto read_w = [&](int s, int h, f32x4 (&v)[FBW]) {
#pragma unroll
      for (int f = 0; f < FBW; ++f) {
        if (IM) {
#pragma unroll
          for (int i = 0; i < 4; ++i) v[f][i] = sb[s][(16 * h + 4 * g + i) * BP + w0 + 16 * f + q16];
        } else {
          v[f] = *reinterpret_cast<const f32x4*>(&sb[s][(w0 + 16 * f + q16) * FKS + 4 * ((4 * h + g) ^ key)]);
        }
      }
    };
    auto read_x = [&](int s, int h, int u) { return *reinterpret_cast<const f32x4*>(&sa[s][(16 * u + q16) * FKS + 4 * ((4 * h + g) ^ key)]); };
    auto multiply = [&](int u, const f32x4 (&v)[FBW]) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int f = 0; f < FBW; ++f) acc[u][f] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[f][i], x[u][i], acc[u][f], 0, 0, 0);
    };
    load(0);
    store(0);
    load(1);  // (K is a multiple of 64)
    __syncthreads();
    for (int kt = 0; kt < KT; ++kt) {
      const int s = kt & 1;
      read_w(s, 0, w[0]);
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = read_x(s, 0, u);
      if (kt + 1 < KT) store(s ^ 1);  // (nobody has read that stage since the last barrier)
      if (kt + 2 < KT) load(kt + 2);
      read_w(s, 1, w[1]);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        multiply(u, w[0]);
        x[u] = read_x(s, 1, u);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) multiply(u, w[1]);
      lds_barrier();
    }
  };
  switch (units) {
    case 1: contract(std::integral_constant<int, (1 < BU ? 1 : BU)>{}); break;
    case 2: contract(std::integral_constant<int, (2 < BU ? 2 : BU)>{}); break;
    case 3: contract(std::integral_constant<int, (3 < BU ? 3 : BU)>{}); break;
    case 4: contract(std::integral_constant<int, (4 < BU ? 4 : BU)>{}); break;
    case 5: contract(std::integral_constant<int, (5 < BU ? 5 : BU)>{}); break;
    case 6: contract(std::integral_constant<int, (6 < BU ? 6 : BU)>{}); break;
    case 7: contract(std::integral_constant<int, (7 < BU ? 7 : BU)>{}); break;
    case 8: contract(std::integral_constant<int, (8 < BU ? 8 : BU)>{}); break;
    case 9: contract(std::integral_constant<int, (9 < BU ? 9 : BU)>{}); break;
    default: contract(std::integral_constant<int, BU>{}); break;
  }
  // lane (q16, g): row q16 of every unit, weight rows 4 g .. 4 g + 3 of every block
#pragma unroll
  for (int f = 0; f < (EPI == F_SWIGLU ? 1 : FBW); ++f) {
    const int nb = EPI == F_SWIGLU ? n0 + wave * 16 : n0 + w0 + 16 * f;
    if (nb < t.nt * OUTF) continue;
    const int n = nb + 4 * g;
    f32x4 b = {0.f, 0.f, 0.f, 0.f};
    if (EPI != F_SWIGLU && bias) b = load4(bias + (size_t)t.expert * N + n);
#pragma unroll
    for (int u = 0; u < BU; ++u) {
      const int r = 16 * u + q16;
      if (r >= t.rows) continue;
      f32x4a4 y;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if constexpr (EPI == F_SWIGLU) y[v] = silu_exact(acc[u][0][v]) * acc[u][FBW - 1][v];
        else if (EPI == F_GELU) y[v] = gelu_exact(acc[u][f][v] + b[v]);
        else y[v] = acc[u][f][v] + b[v];
      }
      *reinterpret_cast<f32x4a4*>(out + (size_t)(t.row0 + r) * N + n) = y;
      if (EPI == F_BIAS && layer.out) {
        const int token = layer.row_map[t.row0 + r];  // (k = 1: the assignment is the token)
        const size_t o = (size_t)token * N + n;
        const float gw = layer.gate_w[token];
        f32x4 a = {0.f, 0.f, 0.f, 0.f};
        if (layer.residual) a = load4(layer.residual + o);
#pragma unroll
        for (int v = 0; v < 4; ++v) a[v] = fmaf(gw, y[v], a[v]);
        *reinterpret_cast<f32x4a4*>(layer.out + o) = a;
      }
    }
  }
  store_share<256>(layer, act, t, n_tiles, K, first_share(layer, act, t, n_tiles, K));
}

// Few tiles: 32 rows x 32 features per workgroup, whose eight wavefronts split the contraction index (runs of 32 values,
// one 128-byte line per row, straight from global memory into MFMA operands); their sums meet in LDS in wavefront
// order.  Bound by latency: a quarter of the tile, an eighth of the chain.
constexpr int SPLIT_WAVES = 8;
template <int EPI, bool IM>
__global__ __launch_bounds__(SPLIT_WAVES * 64) void ffn_f32_split_kernel(
    const float* __restrict__ act, const float* __restrict__ wa, const float* __restrict__ wb, const float* __restrict__ bias,
    const int32_t* __restrict__ offsets, float* __restrict__ out, int E, int N, int K, int n_tiles, F32Layer layer) {
  constexpr int NM = EPI == F_SWIGLU ? 2 : 1;  // weight matrices
  __shared__ float red[SPLIT_WAVES][NM][1024];
  RowTile t;
  if (EPI == F_BIAS && layer.out) fill_rowless_tokens<SPLIT_WAVES>(layer.a2r, offsets[E], layer.T, N, layer.residual, layer.out);
  if (!find_row_tile<32>(offsets, E, n_tiles, t)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const int n0 = t.nt * 32;
  const size_t we = (size_t)t.expert * N * K;
  const float* pa = act + (size_t)act_row(layer, t.row0 + min(l32, t.rows - 1)) * K + 4 * h;
  const float* pw[NM];
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    const float* w = (m ? wb : wa) + we;
    pw[m] = IM ? w + (size_t)(4 * h) * N + n0 + l32 : w + (size_t)(n0 + l32) * K + 4 * h;
  }
  struct Chunk { f32x4 a[4], b[NM][4]; };
  auto load = [&](int c, Chunk& x) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      x.a[kk] = load4(pa + (size_t)c * 32 + 8 * kk);
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        if (IM) {
#pragma unroll
          for (int i = 0; i < 4; ++i) x.b[m][kk][i] = pw[m][(size_t)(c * 32 + 8 * kk + i) * N];
        } else {
          x.b[m][kk] = load4(pw[m] + (size_t)c * 32 + 8 * kk);
        }
      }
    }
  };
  f32x16 acc[NM];
#pragma unroll
  for (int m = 0; m < NM; ++m)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[m][v] = 0.f;
  auto multiply = [&](const Chunk& x) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int m = 0; m < NM; ++m) acc[m] = __builtin_amdgcn_mfma_f32_32x32x2f32(x.a[kk][i], x.b[m][kk][i], acc[m], 0, 0, 0);
  };
  const int n_chunks = K / 32;
  const RowShare share = first_share(layer, act, t, n_tiles, K);
  if (wave < n_chunks) {
    Chunk x[2];
    load(wave, x[0]);
    int c = wave;
    for (; c + SPLIT_WAVES < n_chunks; c += 2 * SPLIT_WAVES) {
      load(c + SPLIT_WAVES, x[1]);
      multiply(x[0]);
      load(min(c + 2 * SPLIT_WAVES, n_chunks - 1), x[0]);
      multiply(x[1]);
    }
    if (c < n_chunks) multiply(x[0]);
  }
#pragma unroll
  for (int m = 0; m < NM; ++m)
#pragma unroll
    for (int v = 0; v < 16; ++v) red[wave][m][v * 64 + lane] = acc[m][v];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 1024 / (SPLIT_WAVES * 64); ++q) {
    const int i = q * SPLIT_WAVES * 64 + tid, v = i >> 6, l = i & 63;
    const int r = (v & 3) + 8 * (v >> 2) + 4 * (l >> 5), n = n0 + (l & 31);
    float u[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      u[m] = red[0][m][i];
#pragma unroll
      for (int w = 1; w < SPLIT_WAVES; ++w) u[m] += red[w][m][i];
    }
    if (r >= t.rows) continue;
    float y = u[0];
    if constexpr (EPI == F_SWIGLU) y = silu_exact(y) * u[NM - 1];
    else {
      if (bias) y += bias[(size_t)t.expert * N + n];
      if (EPI == F_GELU) y = gelu_exact(y);
    }
    out[(size_t)(t.row0 + r) * N + n] = y;
    if (EPI == F_BIAS && layer.out) combine_one(layer, t.row0 + r, N, n, y);
  }
  store_share<SPLIT_WAVES * 64>(layer, act, t, n_tiles, K, share);
}

// Spread of an expert's rows under random routing: Poisson, and routers that like one expert a little more than another
// (random router columns of d values: by about four over the root of 2 d).
double row_sd(double rows) { return std::sqrt(rows + 0.0064 * rows * rows); }
// Row tiles of tm rows that E experts of `rows` rows, at most C each, are expected to have together.
double expected_tiles(int64_t E, int64_t rows, int64_t C, int tm) {
  const double sd = row_sd((double)rows);
  if (sd > tm) return E * (rows / (double)tm + 0.5);
  double t = 1.0;
  for (int64_t i = 1; i * tm < C && i * tm < rows + 5 * sd; ++i) t += 0.5 * std::erfc((i * tm + 0.5 - rows) / (sd * 1.4142135623730951));
  return E * t;
}

// Which kernel (rounds: of 256 CUs):
//  - the kernel that splits the contraction index up to 256 tiles of 64 rows (one for every CU).  Measured (us, 64 rows / split):
//    112 tiles, K 2624: 60 / 50; 144 tiles, K 640: 21 / 18; 256 tiles of 16 rows, K 4096: 99 / 78; 288 tiles, K 2048: 85 / 92;
//    656 tiles, K 448: 38 / 67; 1280 tiles, K 4096: 380 / 548;
//  - 160 rows where long rows meet whole rounds of such tiles (one per CU, or two) that no expert is likely to overflow, since that
//    opens a further round (64 experts of 256 rows, 4096 -> 256, one round: 377 / 580), the features fill their tiles (7 of 339, 5696 ->
//    1472: 413 / 496), and an expert's rows leave its tiles of 64 rows unfilled, or are so many that those do not matter: at 80 to
//    128 rows per tile both multiply the same (32 of 172, 3648 -> 512: 267 / 321);
//  - 80 rows from 256 values on where the tiles come to at most 0.9 of those of 64 rows and fill 0.82 of their rounds, up to the first
//    tiles of the fifth (beyond, up to six, 1.01 on average and a quarter slower), or are more than six rounds, where no single round
//    matters.  One round overflown: 16 experts of 140 rows, 1088 -> 512, 49 / 55; 4.5 rounds: 8 of 1016, 1024 -> 704, 120 / 131.
//    SwiGLU on output-major weights, where the 64-row kernel has two products' weights for half the rows, always but for
//    the start of a second round (1.14); on input-major ones two workgroups fit the LDS of a CU and not three: not in two to three
//    rounds (0.96) nor in four to 5.5 (0.98).
// Over whole layers of random sizes and routing, d_model to 4096, d_ff to 14336, 64 to 16384 tokens, three sets of weights in turn, the
// 362 products that 160 rows serve gain 1.15 over the kernels of 64 rows and the split (five of them lose more than 3 %, by up to 6 %),
// the 1643 that 80 rows serve 1.12 (75, by up to 11 %, mostly where routing takes one tile more than expected).
enum { F32_SPLIT, F32_64, F32_80, F32_160 };
int pick_f32(const moe_config* cfg, int N, int K, bool swiglu, bool input_major) {
  const int64_t rows = (max_rows(cfg) + cfg->E - 1) / cfg->E, E = cfg->E, C = moe_capacity(cfg);
  auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  if (E * up(rows, FM) * up(N, FN) <= 256) return F32_SPLIT;
  const int outf160 = swiglu ? 64 : 128;
  const double most = rows + std::sqrt(2.0 * std::log((double)E)) * row_sd((double)rows);  // of the fullest of E experts
  const int64_t each = up(rows, 160);
  if (K >= 1024 && N >= outf160 && each == up(most < C ? (int64_t)most : C, 160) && up(N, outf160) * outf160 * 20 <= (int64_t)N * 21 &&
      (rows <= 80 * each || rows >= 128 * each)) {
    const double r = E * each * up(N, outf160) / 256.0, pairs = std::ceil(r / 2) * 2;
    if ((r <= 1 && r >= 0.94) || (r > 1 && r >= 0.94 * pairs)) return F32_160;
  }
  const double r80 = expected_tiles(E, rows, C, 80) * up(N, 64) / 256.0, r64 = expected_tiles(E, rows, C, FM) * up(N, FN) / 256.0;
  const bool whole = r80 <= 4.3 && (r80 > 4 || r80 >= 0.82 * std::ceil(r80));
  const bool pays = !swiglu      ? whole || r80 > 6
                    : input_major ? (whole && r80 <= 4 && !(r80 > 2 && r80 <= 3)) || r80 > 5.5
                                  : r80 > 1.65 || (r80 <= 1 && r80 >= 0.8);
  if (K >= 256 && r80 <= 0.9 * r64 && pays) return F32_80;
  return F32_64;
}

template <int EPI, bool IM>
int32_t launch_f32_layout(const moe_config* cfg, const float* act, const float* wa, const float* wb, const float* bias,
                          const int32_t* offsets, float* out, int N, int K, const F32Layer& layer, hipStream_t s) {
  if (max_rows(cfg) == 0) return MOE_OK;
  constexpr bool SW = EPI == F_SWIGLU;
  const int which = pick_f32(cfg, N, K, SW, IM);
  auto run = [&](auto kern, int tm, int tn, int threads) {
    const int n_tiles = (N + tn - 1) / tn;
    const int64_t grid = row_tile_grid(cfg, tm, n_tiles);
    if (grid > INT32_MAX) return fail(MOE_ERR_UNSUPPORTED, "float32 FFN: too many tiles");
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(threads), 0, s, act, wa, wb, bias, offsets, out, cfg->E, N, K, n_tiles, layer);
    return check_hip(hipGetLastError(), "float32 FFN launch");
  };
  switch (which) {
    case F32_SPLIT: return run(ffn_f32_split_kernel<EPI, IM>, 32, 32, SPLIT_WAVES * 64);
    case F32_80: return run(ffn_f32_units_kernel<EPI, IM, SW ? 2 : 1, 5>, 80, 64, 256);
    case F32_160: return run(ffn_f32_units_kernel<EPI, IM, 2, 10>, 160, SW ? 64 : 128, 256);
  }
  return run(ffn_f32_kernel<EPI, IM>, FM, FN, 256);
}

int32_t launch_f32(const moe_config* cfg, int epi, const float* act, const float* wa, const float* wb,
                   const float* bias, const int32_t* offsets, float* out, int N, int K, int layout, const F32Layer& layer, hipStream_t s) {
  const bool im = layout == MOE_LAYOUT_INPUT_MAJOR;
#define MOE_F32_(e) (im ? launch_f32_layout<e, true>(cfg, act, wa, wb, bias, offsets, out, N, K, layer, s) \
                       : launch_f32_layout<e, false>(cfg, act, wa, wb, bias, offsets, out, N, K, layer, s))
  if (epi == F_GELU) return MOE_F32_(F_GELU);
  if (epi == F_SWIGLU) return MOE_F32_(F_SWIGLU);
  return MOE_F32_(F_BIAS);
#undef MOE_F32_
}

// Any shape and alignment: 32 x 32 elements per workgroup, one at a time.
template <typename T>
__global__ __launch_bounds__(256) void transpose_kernel(const T* __restrict__ src, T* __restrict__ dst, int rows, int cols) {
  __shared__ T tile[32][33];
  const size_t base = (size_t)blockIdx.z * rows * cols;
  const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int i = ty; i < 32; i += 8)
    if (r0 + i < rows && c0 + tx < cols) tile[i][tx] = src[base + (size_t)(r0 + i) * cols + c0 + tx];
  __syncthreads();
  for (int i = ty; i < 32; i += 8)
    if (c0 + i < cols && r0 + tx < rows) dst[base + (size_t)(c0 + i) * rows + r0 + tx] = tile[tx][i];
}

// Rows, columns and pointers in whole 16-byte vectors (V elements): 64 x 64 elements per workgroup, 16-byte loads along
// a source row and 16-byte stores along a destination row, so that both sides move whole 128-byte lines (bf16).  HBM
// bound; the 2-byte accesses of the kernel above need eight times the instructions for the same bytes.  The transposition
// itself happens on the way out of LDS, where a thread collects V elements of one column; an LDS row is padded by one
// dword, which puts the eight row groups that a wavefront reads at once on different banks.  Measured on MI355X, 16 bf16
// matrices of 4096 x 1024: 121 us with the kernel above, 40 us with this one (6.7 TB/s of reads and writes); 8 of
// 14336 x 4096, which no cache holds: 368 us (5.1 TB/s).
template <typename T>
__global__ __launch_bounds__(256) void transpose_vec_kernel(const T* __restrict__ src, T* __restrict__ dst, int rows, int cols) {
  constexpr int V = 16 / sizeof(T), N = 64, CH = N / V;  // elements per vector, tile edge, vectors per tile row
  constexpr int PITCH = N + 4 / sizeof(T);
  __shared__ __attribute__((aligned(16))) T tile[N * PITCH];
  const size_t base = (size_t)blockIdx.z * rows * cols;
  const int c0 = blockIdx.x * N, r0 = blockIdx.y * N;
  uint4 v[N * CH / 256];
#pragma unroll
  for (int q = 0; q < N * CH / 256; ++q) {
    const int i = q * 256 + threadIdx.x, r = i / CH, c = (i % CH) * V;
    v[q] = uint4{0u, 0u, 0u, 0u};
    if (r0 + r < rows && c0 + c < cols) v[q] = *reinterpret_cast<const uint4*>(src + base + (size_t)(r0 + r) * cols + c0 + c);
  }
#pragma unroll
  for (int q = 0; q < N * CH / 256; ++q) {
    const int i = q * 256 + threadIdx.x, r = i / CH, c = (i % CH) * V;
    uint32_t* p = reinterpret_cast<uint32_t*>(tile + r * PITCH + c);  // (a padded row starts on a dword, not on 16 bytes)
    p[0] = v[q].x; p[1] = v[q].y; p[2] = v[q].z; p[3] = v[q].w;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < N * CH / 256; ++q) {
    const int i = q * 256 + threadIdx.x, c = i / CH, r = (i % CH) * V;  // destination row c, elements r .. r + V - 1
    T o[V];
#pragma unroll
    for (int j = 0; j < V; ++j) o[j] = tile[(r + j) * PITCH + c];
    if (c0 + c < cols && r0 + r < rows) {
      uint4 w;
      __builtin_memcpy(&w, o, 16);
      *reinterpret_cast<uint4*>(dst + base + (size_t)(c0 + c) * rows + r0 + r) = w;
    }
  }
}

template <typename T>
void launch_transpose(const void* src, void* dst, int E, int rows, int cols, hipStream_t s) {
  constexpr int V = 16 / sizeof(T);
  const bool vec = rows % V == 0 && cols % V == 0 && (((uintptr_t)src | (uintptr_t)dst) & 15) == 0;
  const int n = vec ? 64 : 32;
  const dim3 grid((cols + n - 1) / n, (rows + n - 1) / n, E), block(256);
  if (vec) hipLaunchKernelGGL(transpose_vec_kernel<T>, grid, block, 0, s, (const T*)src, (T*)dst, rows, cols);
  else hipLaunchKernelGGL(transpose_kernel<T>, grid, block, 0, s, (const T*)src, (T*)dst, rows, cols);
}

__global__ void clear_ints_kernel(int32_t* p, int n) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0;
}

}  // namespace

int32_t launch_gemm1(const moe_config* cfg, const moe_weights* w, const void* xd, const int32_t* offsets, void* h,
                     const int32_t* row_map, int32_t* tile_counters, hipStream_t s, void* xd_out) {
  if (cfg->dtype == MOE_BF16) return launch_gemm1_bf16(cfg, w, xd, offsets, h, row_map, tile_counters, s);
  if (!row_map != !xd_out) return fail(MOE_ERR_INVALID_ARG, "float32 FFN: a gathering product stores the dispatched rows");
  const F32Layer layer = {row_map, (float*)xd_out, nullptr, nullptr, nullptr, nullptr, cfg->T};
  if (cfg->act == MOE_ACT_SWIGLU)
    return launch_f32(cfg, F_SWIGLU, (const float*)xd, (const float*)w->w_gate_proj, (const float*)w->w_up, nullptr,
                      offsets, (float*)h, cfg->d_ff, cfg->d_model, w->layout, layer, s);
  return launch_f32(cfg, F_GELU, (const float*)xd, (const float*)w->w1, nullptr, (const float*)w->b1, offsets,
                    (float*)h, cfg->d_ff, cfg->d_model, w->layout, layer, s);
}

int32_t launch_gemm2(const moe_config* cfg, const moe_weights* w, const void* h, const int32_t* offsets, void* yd,
                     int32_t* tile_counters, hipStream_t s) {
  if (cfg->dtype == MOE_BF16) return launch_gemm2_bf16(cfg, w, h, offsets, yd, tile_counters, s);
  const bool sw = cfg->act == MOE_ACT_SWIGLU;
  return launch_f32(cfg, F_BIAS, (const float*)h, (const float*)(sw ? w->w_down : w->w2), nullptr,
                    (const float*)(sw ? nullptr : w->b2), offsets, (float*)yd, cfg->d_model, cfg->d_ff, w->layout, F32Layer{}, s);
}

// With one expert per token a dispatched row is the only term of its token's output, so the second GEMM can
// finish the combine itself; in bf16 it then stores no yd (a workspace has no such segment), in float32 it does.
bool gemm2_can_combine(const moe_config* cfg) { return cfg->dtype == MOE_BF16 && cfg->k == 1; }

int32_t launch_gemm2_combine(const moe_config* cfg, const moe_weights* w, const void* h, const int32_t* offsets,
                             const int32_t* r2a, const float* topk_w, const void* residual, void* out,
                             const int32_t* a2r, int32_t* tile_counters, hipStream_t s, void* yd) {
  if (cfg->k != 1) return fail(MOE_ERR_UNSUPPORTED, "combine in the second GEMM needs k = 1");
  if (cfg->dtype == MOE_BF16) return launch_gemm2_combine_bf16(cfg, w, h, offsets, r2a, topk_w, residual, out, a2r, tile_counters, s);
  const bool sw = cfg->act == MOE_ACT_SWIGLU;
  const F32Layer layer = {r2a, nullptr, topk_w, (const float*)residual, (float*)out, a2r, cfg->T};
  return launch_f32(cfg, F_BIAS, (const float*)h, (const float*)(sw ? w->w_down : w->w2), nullptr,
                    (const float*)(sw ? nullptr : w->b2), offsets, (float*)yd, cfg->d_model, cfg->d_ff, w->layout, layer, s);
}

}  // namespace moesys

using namespace moesys;

extern "C" int32_t moe_expert_ffn(const moe_config* cfg, const moe_weights* w, const void* xd,
                                  const int32_t* expert_offsets, void* yd, void* ws, size_t ws_bytes, void* stream) {
  int32_t st = moe_config_check(cfg);
  if (st != MOE_OK) return st;
  st = check_weights(cfg, w);
  if (st != MOE_OK) return st;
  if (!expert_offsets) return fail(MOE_ERR_INVALID_ARG, "moe_expert_ffn: expert_offsets is NULL");
  const size_t need = moe_workspace_bytes(cfg, MOE_WS_FFN);
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < need)
    return fail(MOE_ERR_WORKSPACE, "moe_expert_ffn: workspace needs %zu bytes, 256-byte aligned (got %zu)", need, ws_bytes);
  if (max_rows(cfg) > 0 && (!xd || !yd)) return fail(MOE_ERR_INVALID_ARG, "moe_expert_ffn: xd and yd must be non-NULL");
  // the tile counters sit behind h; nothing ran before us on this workspace, so clear the first GEMM's here
  int32_t* ctr = (int32_t*)((char*)ws + ffn_counter_offset(cfg));
  if (cfg->dtype == MOE_BF16) {
    hipLaunchKernelGGL(clear_ints_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, ctr, 8);
    if ((st = check_hip(hipGetLastError(), "counter clear launch")) != MOE_OK) return st;
  }
  st = launch_gemm1(cfg, w, xd, expert_offsets, ws, nullptr, ctr, (hipStream_t)stream);
  if (st != MOE_OK) return st;
  return launch_gemm2(cfg, w, ws, expert_offsets, yd, ctr, (hipStream_t)stream);
}

extern "C" int32_t moe_transpose_expert_weights(const void* src, void* dst, int32_t E, int32_t rows, int32_t cols,
                                                int32_t dtype, void* stream) {
  if (!src || !dst || src == dst) return fail(MOE_ERR_INVALID_ARG, "moe_transpose_expert_weights: src/dst NULL or aliased");
  if (E < 1 || rows < 1 || cols < 1 || E > 65535) return fail(MOE_ERR_INVALID_ARG, "moe_transpose_expert_weights: bad shape");
  if (dtype != MOE_F32 && dtype != MOE_BF16) return fail(MOE_ERR_INVALID_ARG, "moe_transpose_expert_weights: dtype unknown");
  if ((rows + 31) / 32 > 65535) return fail(MOE_ERR_UNSUPPORTED, "moe_transpose_expert_weights: rows too large");
  if (dtype == MOE_BF16) launch_transpose<uint16_t>(src, dst, E, rows, cols, (hipStream_t)stream);
  else launch_transpose<float>(src, dst, E, rows, cols, (hipStream_t)stream);
  return check_hip(hipGetLastError(), "transpose launch");
}

// Rows per tile of the kernel that serves the float32 experts' first (which = 0) or second (1) product, + 2 for input-major weights;
// 32: the one that splits the contraction index.  For the tests of the rule above; host only, not part of the interface in moesys.h.
extern "C" int32_t moe_test_f32_tile_rows(const moe_config* cfg, int32_t which) {
  using namespace moesys;
  if (moe_config_check(cfg) != MOE_OK || cfg->dtype != MOE_F32) return 0;
  const bool second = which & 1;
  const int N = second ? cfg->d_model : cfg->d_ff, K = second ? cfg->d_ff : cfg->d_model;
  const int rows[] = {32, FM, 80, 160};
  return rows[pick_f32(cfg, N, K, !second && cfg->act == MOE_ACT_SWIGLU, which & 2)];
}
