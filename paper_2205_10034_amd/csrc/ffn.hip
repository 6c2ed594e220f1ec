// Expert FFN entry point, the float32 grouped GEMM (correctness configuration)
// and the one-time expert weight transpose.
//
// The bf16 MFMA grouped GEMM lives in grouped_gemm_bf16.hip; the float32 path
// below multiplies on the float32 matrix instructions.
#include "moesys_internal.h"
#include "row_tiles.h"

namespace moesys {

int32_t launch_gemm1_bf16(const moe_config*, const moe_weights*, const void*, const int32_t*, void*, const int32_t*, int32_t*,
                          hipStream_t);
int32_t launch_gemm2_bf16(const moe_config*, const moe_weights*, const void*, const int32_t*, void*, int32_t*, hipStream_t);
int32_t launch_gemm2_combine_bf16(const moe_config*, const moe_weights*, const void*, const int32_t*, const int32_t*,
                                  const float*, const void*, void*, int32_t*, hipStream_t);

namespace {

enum { F_GELU = 0, F_SWIGLU = 1, F_BIAS = 2 };

__device__ __forceinline__ float gelu_exact(float u) { return 0.5f * u * (1.f + erff(u * 0.70710678118654752f)); }
__device__ __forceinline__ float silu_exact(float u) { return u / (1.f + expf(-u)); }

// Four floats from any float address (one 16-byte load; the hardware asks for no more than 4-byte alignment).
typedef float f32x4a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
__device__ __forceinline__ f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4a4*>(p); }

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
                                                         int N, int K, int n_tiles) {
  constexpr int NB = EPI == F_SWIGLU ? 2 : 1;          // 32-feature blocks per wavefront
  constexpr int TN = FN * NB;                          // weight rows per tile
  constexpr int BP = IM ? TN + 4 : FPITCH, BROWS = IM ? FKS : TN;
  __shared__ __attribute__((aligned(16))) float sa[2][FM * FPITCH];
  __shared__ __attribute__((aligned(16))) float sb[2][BROWS * BP];
  RowTile t;
  if (!find_row_tile<FM>(offsets, E, n_tiles, t)) return;
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
    pa[q] = act + (size_t)(t.row0 + min(r, t.rows - 1)) * K + 4 * c;
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
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int r = wm * 32 + (v & 3) + 8 * (v >> 2) + 4 * h;
    if (r >= t.rows) continue;
    float u = acc[0][v];
    if constexpr (EPI == F_SWIGLU) u = silu_exact(u) * acc[NB - 1][v];
    else if (EPI == F_GELU) u = gelu_exact(u + b);
    else u += b;
    out[(size_t)(t.row0 + r) * N + n] = u;
  }
}

// Few tiles: 32 rows x 32 features per workgroup, whose eight wavefronts split the contraction index (runs of 32 values,
// one 128-byte line per row, straight from global memory into MFMA operands); their sums meet in LDS in wavefront
// order.  Bound by latency: a quarter of the tile, an eighth of the chain.
constexpr int SPLIT_WAVES = 8;
template <int EPI, bool IM>
__global__ __launch_bounds__(SPLIT_WAVES * 64) void ffn_f32_split_kernel(
    const float* __restrict__ act, const float* __restrict__ wa, const float* __restrict__ wb, const float* __restrict__ bias,
    const int32_t* __restrict__ offsets, float* __restrict__ out, int E, int N, int K, int n_tiles) {
  constexpr int NM = EPI == F_SWIGLU ? 2 : 1;  // weight matrices
  __shared__ float red[SPLIT_WAVES][NM][1024];
  RowTile t;
  if (!find_row_tile<32>(offsets, E, n_tiles, t)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const int n0 = t.nt * 32;
  const size_t we = (size_t)t.expert * N * K;
  const float* pa = act + (size_t)(t.row0 + min(l32, t.rows - 1)) * K + 4 * h;
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
  }
}

template <int EPI, bool IM>
int32_t launch_f32_layout(const moe_config* cfg, const float* act, const float* wa, const float* wb, const float* bias,
                          const int32_t* offsets, float* out, int N, int K, hipStream_t s) {
  const int64_t rmax = max_rows(cfg);
  if (rmax == 0) return MOE_OK;
  // The 64-row kernel from 257 tiles on (one for every CU), for evenly loaded experts; below, the kernel that splits the
  // contraction index.  Measured (us, 64 rows / split): 112 tiles, K 2624: 60 / 50; 144 tiles, K 640: 21 / 18; 256 tiles of
  // 16 rows, K 4096: 99 / 78; 288 tiles, K 2048: 85 / 92; 656 tiles, K 448: 38 / 67; 1280 tiles, K 4096: 380 / 548.
  const int64_t rows_each = (rmax + cfg->E - 1) / cfg->E;
  const bool split = cfg->E * ((rows_each + FM - 1) / FM) * ((N + FN - 1) / FN) <= 256;
  const int tm = split ? 32 : FM, tn = split ? 32 : FN;
  const int64_t grid = row_tile_grid(cfg, tm, (N + tn - 1) / tn);
  if (grid > INT32_MAX) return fail(MOE_ERR_UNSUPPORTED, "float32 FFN: too many tiles");
  const dim3 g((unsigned)grid);
  const int n_tiles = (N + tn - 1) / tn;
  if (split)
    hipLaunchKernelGGL((ffn_f32_split_kernel<EPI, IM>), g, dim3(SPLIT_WAVES * 64), 0, s, act, wa, wb, bias, offsets, out, cfg->E, N, K, n_tiles);
  else
    hipLaunchKernelGGL((ffn_f32_kernel<EPI, IM>), g, dim3(256), 0, s, act, wa, wb, bias, offsets, out, cfg->E, N, K, n_tiles);
  return check_hip(hipGetLastError(), "float32 FFN launch");
}

int32_t launch_f32(const moe_config* cfg, int epi, const float* act, const float* wa, const float* wb,
                   const float* bias, const int32_t* offsets, float* out, int N, int K, int layout, hipStream_t s) {
  const bool im = layout == MOE_LAYOUT_INPUT_MAJOR;
#define MOE_F32_(e) (im ? launch_f32_layout<e, true>(cfg, act, wa, wb, bias, offsets, out, N, K, s) \
                       : launch_f32_layout<e, false>(cfg, act, wa, wb, bias, offsets, out, N, K, s))
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
                     const int32_t* row_map, int32_t* tile_counters, hipStream_t s) {
  if (cfg->dtype == MOE_BF16) return launch_gemm1_bf16(cfg, w, xd, offsets, h, row_map, tile_counters, s);
  if (row_map) return fail(MOE_ERR_UNSUPPORTED, "float32 FFN reads dispatched rows only");
  if (cfg->act == MOE_ACT_SWIGLU)
    return launch_f32(cfg, F_SWIGLU, (const float*)xd, (const float*)w->w_gate_proj, (const float*)w->w_up, nullptr,
                      offsets, (float*)h, cfg->d_ff, cfg->d_model, w->layout, s);
  return launch_f32(cfg, F_GELU, (const float*)xd, (const float*)w->w1, nullptr, (const float*)w->b1, offsets,
                    (float*)h, cfg->d_ff, cfg->d_model, w->layout, s);
}

int32_t launch_gemm2(const moe_config* cfg, const moe_weights* w, const void* h, const int32_t* offsets, void* yd,
                     int32_t* tile_counters, hipStream_t s) {
  if (cfg->dtype == MOE_BF16) return launch_gemm2_bf16(cfg, w, h, offsets, yd, tile_counters, s);
  const bool sw = cfg->act == MOE_ACT_SWIGLU;
  return launch_f32(cfg, F_BIAS, (const float*)h, (const float*)(sw ? w->w_down : w->w2), nullptr,
                    (const float*)(sw ? nullptr : w->b2), offsets, (float*)yd, cfg->d_model, cfg->d_ff, w->layout, s);
}

// With one expert per token a dispatched row is the only term of its token's output, so the second GEMM can
// finish the combine itself (bf16 only).
bool gemm2_can_combine(const moe_config* cfg) { return cfg->dtype == MOE_BF16 && cfg->k == 1; }

int32_t launch_gemm2_combine(const moe_config* cfg, const moe_weights* w, const void* h, const int32_t* offsets,
                             const int32_t* r2a, const float* topk_w, const void* residual, void* out,
                             int32_t* tile_counters, hipStream_t s) {
  if (!gemm2_can_combine(cfg)) return fail(MOE_ERR_UNSUPPORTED, "combine in the second GEMM needs bf16 and k = 1");
  return launch_gemm2_combine_bf16(cfg, w, h, offsets, r2a, topk_w, residual, out, tile_counters, s);
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
