// Expert FFN products for steps of very few tokens (k*T <= 8 assignments in all, so no expert has more rows
// than that; up to 16 where the weight-streaming kernels do not serve): the single-request end of the paper's
// inference scenario (Section 3.3, batch size 1).
//
//   out[r, n] = epilogue( sum_k act[r, k] * W_e[n, k] )      for the rows r of every expert e that has any
//
// With one or two rows per activated expert the product is a matrix-vector product: its time is the time to
// stream the activated experts' weights once, and the MFMA tiles of the grouped GEMM (256 output features per
// workgroup) leave most CUs without work: 2 experts x N/256 tiles.  Here a wavefront owns FPW weight rows
// and its 64 lanes split the contraction index (16 bytes per lane and row: every weight row is read with
// wave-wide contiguous 1 KB loads, FPW of them in flight per wavefront and K block), keeps the partial sums
// of its weight rows x the expert's rows in registers, and adds them across the lanes at the end (a fixed
// butterfly: results do not depend on scheduling).  Workgroup (bx, r0) serves the expert whose FIRST row is
// dispatched row r0 and exits if there is none, so the grid needs no list of the activated experts.  Two shapes
// (the FPW x ROWS partial sums must fit the registers): 8 weight rows x up to 8 rows, 4 x up to 16.  With 9 to 16
// assignments the weight-streaming MFMA kernels (expert_stream_bf16.hip) are faster: 16 assignments over 64 experts of
// 2048 x 8192 118 + 111 us here, 99 + 95 there; with 8 assignments 56 + 52 here, 58 + 57 there.  The 4 x 16 shape serves
// what those kernels leave: contraction lengths beyond their 32-bit offsets, and calls whose tuning keys keep them out.
#include "gate_rank.h"
#include "moesys_internal.h"
#include "wave_util.h"

namespace moesys {

bool expert_stream_applies(const moe_config* cfg, int N, int K, int epi);

namespace {

constexpr int GV_MAX_ROWS = 16;  // rows of one expert, at most (= assignments of the whole step)
constexpr int GV_WAVES = 4;
constexpr int RANKED_SLICES = 16;  // slices of partial logits that expert_gemv_ranked_kernel adds, at most

// NT: non-temporal (nobody else reads a weight, and the call's weights exceed the last-level cache, weights_exceed_cache)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <bool NT>
__device__ __forceinline__ uint4 load_weights(const uint16_t* p) {
  if constexpr (!NT) return *reinterpret_cast<const uint4*>(p);
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return uint4{v.x, v.y, v.z, v.w};
}

enum GvEpi { GV_GELU = 0, GV_SWIGLU = 1, GV_BIAS = 2, GV_COMBINE = 3 };

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float lo16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi16(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ uint16_t bf16_of(float v) {  // round to nearest even
  return (uint16_t)(__builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{v, 0.f}, bf16x2)) & 0xffffu);
}
__device__ __forceinline__ float gelu_exact(float u) { return 0.5f * u * erfcf(-u * 0.70710678118654752f); }

// What the kernels below share, so that a product has the same bits in each: eight terms in order, the sum over the lanes (in every
// lane), the end of the first product (u: the up projection's sum, b: the bias).
struct Row8 { float v[8]; };
__device__ __forceinline__ Row8 unpack8(const uint4& x) {
  return Row8{{lo16(x.x), hi16(x.x), lo16(x.y), hi16(x.y), lo16(x.z), hi16(x.z), lo16(x.w), hi16(x.w)}};
}
__device__ __forceinline__ float add8(float a, const uint4& w, const Row8& x) {
  a = fmaf(lo16(w.x), x.v[0], a); a = fmaf(hi16(w.x), x.v[1], a);
  a = fmaf(lo16(w.y), x.v[2], a); a = fmaf(hi16(w.y), x.v[3], a);
  a = fmaf(lo16(w.z), x.v[4], a); a = fmaf(hi16(w.z), x.v[5], a);
  a = fmaf(lo16(w.w), x.v[6], a); a = fmaf(hi16(w.w), x.v[7], a);
  return a;
}
__device__ __forceinline__ float sum_lanes(float v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}
template <int EPI>
__device__ __forceinline__ float first_end(float v, float u, float b) {
  return EPI == GV_SWIGLU ? v * __builtin_amdgcn_rcpf(1.f + __expf(-v)) * u : gelu_exact(v + b);
}

// EPI: GV_GELU out = gelu(. + bias); GV_SWIGLU out = silu(. Wg) * (. Wu) (a wavefront's weight rows are
// FPW/2 of Wg and the same FPW/2 of Wu); GV_BIAS out = . + bias; GV_COMBINE (k = 1) out[token] =
// residual[token] + gate_w[token] * (. + bias) with token = row_map[r].
// GATHER: act is x[T, K] and row r reads token row_map[r] mod T.
// KSPLIT: the four wavefronts of a workgroup share one set of GV_FPW weight rows and split the contraction index
// (their sums meet in LDS, in wavefront order): four times the workgroups, for long rows and few experts.
template <int EPI, bool GATHER, int GV_ROWS, int GV_FPW, bool KSPLIT, bool NT>
__global__ __launch_bounds__(GV_WAVES * 64) void expert_gemv_kernel(
    const uint16_t* __restrict__ act, const uint16_t* __restrict__ wa, const uint16_t* __restrict__ wb,
    const uint16_t* __restrict__ bias, const int32_t* __restrict__ offsets, uint16_t* out,
    const int32_t* __restrict__ row_map, const float* __restrict__ gate_w, const uint16_t* residual,
    const int32_t* __restrict__ a2r, const int64_t* __restrict__ eoff, int T, int E, int N, int K, int reps) {
  constexpr int OUTF = EPI == GV_SWIGLU ? GV_FPW / 2 : GV_FPW;  // output features per wavefront
  __shared__ int s_e;
  __shared__ float red[KSPLIT ? GV_WAVES : 1][GV_ROWS][GV_FPW];
  const int r0 = blockIdx.y;
  if (threadIdx.x == 0) s_e = -1;
  __syncthreads();
  for (int e = threadIdx.x; e < E; e += GV_WAVES * 64)
    if (offsets[e] == r0 && offsets[e + 1] > r0) s_e = e;  // at most one expert starts at row r0
  __syncthreads();
  const int e = s_e;
  if constexpr (EPI == GV_COMBINE) fill_rowless_tokens<GV_WAVES>(a2r, offsets[E], T, N, residual, out);
  if (e < 0) return;
  const int rows = min(offsets[e + 1] - r0, GV_ROWS);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t wbase = eoff ? eoff[e] : (int64_t)e * N * K;
  const uint16_t* xrow[GV_ROWS];
  int token[GV_ROWS];
#pragma unroll
  for (int r = 0; r < GV_ROWS; ++r) {
    const int rr = r0 + min(r, rows - 1);  // (rows past the expert's last re-read it; their sums are not used)
    int src = rr;
    token[r] = 0;
    if (GATHER || EPI == GV_COMBINE) {
      int t = row_map[rr];
      while (t >= T) t -= T;  // assignment id j*T + t -> token (j < k <= 8)
      token[r] = t;
      if (GATHER) src = t;
    }
    xrow[r] = act + (int64_t)src * K;
  }

  // a workgroup works through `reps` consecutive blocks of output features (with a short contraction index one
  // block is too little work per workgroup)
  for (int rep = 0; rep < reps; ++rep) {
    // first output feature of this wavefront
    const int n0 = KSPLIT ? (blockIdx.x * reps + rep) * OUTF : ((blockIdx.x * reps + rep) * GV_WAVES + wave) * OUTF;
    const uint16_t* wrow[GV_FPW];
#pragma unroll
    for (int j = 0; j < GV_FPW; ++j) {
      if (EPI == GV_SWIGLU) wrow[j] = (j < OUTF ? wa : wb) + wbase + (int64_t)(n0 + j % OUTF) * K;
      else wrow[j] = wa + wbase + (int64_t)(n0 + j) * K;
    }
    float acc[GV_FPW][GV_ROWS];
  #pragma unroll
    for (int j = 0; j < GV_FPW; ++j)
  #pragma unroll
      for (int r = 0; r < GV_ROWS; ++r) acc[j][r] = 0.f;

    for (int kb = (KSPLIT ? (int)threadIdx.x : lane) * 8; kb < K; kb += (KSPLIT ? GV_WAVES : 1) * 64 * 8) {
      uint4 wv[GV_FPW], xv[GV_ROWS];
  #pragma unroll
      for (int j = 0; j < GV_FPW; ++j) wv[j] = load_weights<NT>(wrow[j] + kb);
  #pragma unroll
      for (int r = 0; r < GV_ROWS; ++r)
        if (r < rows) xv[r] = *reinterpret_cast<const uint4*>(xrow[r] + kb);
  #pragma unroll
      for (int r = 0; r < GV_ROWS; ++r) {
        if (r < rows) {  // (wave-uniform)
          const Row8 x = unpack8(xv[r]);
  #pragma unroll
          for (int j = 0; j < GV_FPW; ++j) acc[j][r] = add8(acc[j][r], wv[j], x);
        }
      }
    }

    // sums over the lanes; afterwards every lane holds every total
  #pragma unroll
    for (int r = 0; r < GV_ROWS; ++r) {
      if (r < rows) {
  #pragma unroll
        for (int j = 0; j < GV_FPW; ++j) acc[j][r] = sum_lanes(acc[j][r]);
      }
    }

    if constexpr (KSPLIT) {  // the wavefronts' sums meet: lane j < GV_FPW carries weight row j
      if (rep) __syncthreads();  // (the previous block's sums have been read)
#pragma unroll
      for (int r = 0; r < GV_ROWS; ++r) {
        if (r < rows && lane < GV_FPW) {
          float v = acc[0][r];
#pragma unroll
          for (int j = 1; j < GV_FPW; ++j) v = lane == j ? acc[j][r] : v;
          red[wave][r][lane] = v;
        }
      }
      __syncthreads();
      if (wave == 0 && lane < GV_FPW) {
#pragma unroll
        for (int r = 0; r < GV_ROWS; ++r) {
          if (r < rows) {
            float v = red[0][r][lane];
#pragma unroll
            for (int w = 1; w < GV_WAVES; ++w) v += red[w][r][lane];
            red[0][r][lane] = v;  // (only this lane reads and writes the element)
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < GV_ROWS; ++r)
        if (r < rows)
#pragma unroll
          for (int j = 0; j < GV_FPW; ++j) acc[j][r] = red[0][r][j];  // every lane holds every total again
    }
    // lane j < OUTF finishes output feature n0 + j of every row
    if ((!KSPLIT || wave == 0) && lane < OUTF) {
      const int n = n0 + lane;
      float b = 0.f;
      if (EPI != GV_SWIGLU && bias) b = lo16((uint32_t)bias[(eoff ? eoff[e] : (int64_t)e * N) + n]);  // (eoff: as for the weights)
  #pragma unroll
      for (int r = 0; r < GV_ROWS; ++r) {
        if (r < rows) {
          float v = acc[0][r], u = 0.f;
  #pragma unroll
          for (int j = 1; j < OUTF; ++j) v = lane == j ? acc[j][r] : v;
          if (EPI == GV_SWIGLU) {
            u = acc[OUTF][r];
  #pragma unroll
            for (int j = 1; j < OUTF; ++j) u = lane == j ? acc[OUTF + j][r] : u;
          }
          if (EPI == GV_SWIGLU || EPI == GV_GELU) v = first_end<EPI>(v, u, b);
          else v += b;
          if (EPI == GV_COMBINE) {
            const size_t o = (size_t)token[r] * N + n;
            const float res = residual ? lo16((uint32_t)residual[o]) : 0.f;
            out[o] = bf16_of(fmaf(gate_w[token[r]], v, res));
          } else {
            out[(size_t)(r0 + r) * N + n] = bf16_of(v);
          }
        }
      }
    }
  }
}

// Ranks the token of a one-token step from its partial logits, in every wavefront; returns the selected experts, bit e for expert e.
// write: the workgroup writes the routing tables.
__device__ __forceinline__ unsigned long long rank_one_token(const double* __restrict__ part, int slices, const float* __restrict__ br, int renorm,
                                                             int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                                             int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                                             int32_t* __restrict__ a2r, int32_t* __restrict__ r2a,
                                                             int32_t* __restrict__ clear8, int E, int k, bool write) {
  __shared__ double zs[GV_WAVES][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int sel;  // lane j < k: the j-th selection (every wavefront ranks for itself)
  float sel_w;
  {
    double v[RANKED_SLICES / GV_WAVES], z = 0.0;
#pragma unroll
    for (int q = 0; q < RANKED_SLICES / GV_WAVES; ++q)
      v[q] = part[(size_t)min(q * GV_WAVES + wave, slices - 1) * E + min(lane, E - 1)];
#pragma unroll
    for (int q = 0; q < RANKED_SLICES / GV_WAVES; ++q) z += q * GV_WAVES + wave < slices ? v[q] : 0.0;
    zs[wave][lane] = z;
    __syncthreads();
    const int e = min(lane, E - 1);
    z = zs[0][e] + zs[1][e] + zs[2][e] + zs[3][e] + (br ? (double)br[e] : 0.0);
    static_assert(GV_WAVES == 4, "four partial sums");
    sel = rank_wave(lane < E ? z : -INFINITY, lane, E, k, renorm, sel_w);
  }
  unsigned long long chosen = 0;  // bit e: expert e selected; a selection that is no expert (NaN logits) gets no row
  for (int j = 0; j < k; ++j) {
    const int e = valid_expert(__builtin_amdgcn_readlane(sel, j), E);
    if (e >= 0) chosen |= 1ull << e;
  }
  if (write && wave == 0) {
    if (lane < E) {
      counts[lane] = (int)((chosen >> lane) & 1ull);
      offsets[lane] = __popcll(chosen & ((1ull << lane) - 1ull));
    }
    if (lane == 0) offsets[E] = __popcll(chosen);
    if (lane < k) {
      const int e = valid_expert(sel, E), row = e >= 0 ? __popcll(chosen & ((1ull << e) - 1ull)) : -1;
      topk_idx[lane] = sel;
      topk_w[lane] = sel_w;
      a2r[lane] = row;
      if (row >= 0) r2a[row] = lane;
    }
    if (lane < 8) clear8[lane] = 0;
  }
  return chosen;
}

// The same alone, for a caller that routes and runs the experts in two calls: the same bits as below.
__global__ __launch_bounds__(GV_WAVES * 64) void rank_one_token_kernel(const double* __restrict__ part, int slices, const float* __restrict__ br,
                                                                      int renorm, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                                                      int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                                                      int32_t* __restrict__ a2r, int32_t* __restrict__ r2a,
                                                                      int32_t* __restrict__ clear8, int E, int k) {
  rank_one_token(part, slices, br, renorm, topk_idx, topk_w, counts, offsets, a2r, r2a, clear8, E, k, true);
}

// A step of ONE token: ranking, routing tables and the first product in one kernel.  The router's partial logits (float64, E
// values per slice of the contraction index) are a few KB in L2: every workgroup adds them in slice order and ranks the token by
// itself, so that the product starts at the experts' weights where a kernel of its own would rank first and the product then
// walk offsets -> row -> token -> weights; workgroup (0, 0) writes the tables that the second product reads.  Row r is the r-th
// selected expert in expert order and there is one row per expert, so the sums of two 1 KB pieces of FPW weight rows fit the
// registers at once.  E <= 64.  Measured on MI355X, 64 experts 2048 x 8192, k 2: ranking kernel 5.6 us + product 19.5, now 18.6 together;
// whole one-token layers (us, before / now, the wider combine kernel below included): that one 45.3 / 37.4; 16 experts 1792 x 2816
// 25.8 / 16.8; 24 of 1536 x 4096, k 4 42.1 / 28.0; 8 SwiGLU of 4096 x 14336 127 / 119.
// KSPLIT: as in the kernel above and by the same rule, so that a sum has the same terms in the same order in both.  Whole layers (us,
// never split / split): 8 experts 4096 x 2048 20.8 / 20.2, 4096 x 7168 50.8 / 48.7, SwiGLU 4096 x 3584 41.6 / 38.5.
template <int EPI, int FPW, bool NT, bool KSPLIT>
__global__ __launch_bounds__(GV_WAVES * 64) void expert_gemv_ranked_kernel(
    const uint16_t* __restrict__ x, const double* __restrict__ part, int slices, const float* __restrict__ br, int renorm,
    const uint16_t* __restrict__ wa, const uint16_t* __restrict__ wb, const uint16_t* __restrict__ bias, uint16_t* __restrict__ out,
    const int64_t* __restrict__ eoff, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w, int32_t* __restrict__ counts,
    int32_t* __restrict__ offsets, int32_t* __restrict__ a2r, int32_t* __restrict__ r2a, int32_t* __restrict__ clear8, int E, int N,
    int K, int k) {
  constexpr int OUTF = EPI == GV_SWIGLU ? FPW / 2 : FPW;  // output features per wavefront (KSPLIT: per workgroup)
  constexpr int PIECE = (KSPLIT ? GV_WAVES : 1) * 64 * 8;
  __shared__ float red[KSPLIT ? GV_WAVES : 1][FPW];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  unsigned long long chosen = rank_one_token(part, slices, br, renorm, topk_idx, topk_w, counts, offsets, a2r, r2a, clear8, E, k,
                                             blockIdx.x == 0 && blockIdx.y == 0);
  const int row = blockIdx.y;
  if (row >= __popcll(chosen)) return;
  for (int r = 0; r < row; ++r) chosen &= chosen - 1;
  const int e = __builtin_ctzll(chosen);
  const int64_t wbase = eoff ? eoff[e] : (int64_t)e * N * K;
  const int n0 = (KSPLIT ? (int)blockIdx.x : (int)blockIdx.x * GV_WAVES + wave) * OUTF;  // first output feature of this wavefront
  const uint16_t* wrow[FPW];
#pragma unroll
  for (int j = 0; j < FPW; ++j)
    wrow[j] = (EPI == GV_SWIGLU && j >= OUTF ? wb : wa) + wbase + (int64_t)(n0 + j % OUTF) * K;
  float acc[FPW];
#pragma unroll
  for (int j = 0; j < FPW; ++j) acc[j] = 0.f;
  auto add = [&](const uint4 (&wv)[FPW], const uint4& xv) {
    const Row8 x8 = unpack8(xv);
#pragma unroll
    for (int j = 0; j < FPW; ++j) acc[j] = add8(acc[j], wv[j], x8);
  };
  for (int kb = (KSPLIT ? (int)threadIdx.x : lane) * 8; kb < K; kb += 2 * PIECE) {
    const bool two = kb + PIECE < K;
    const int kb2 = two ? kb + PIECE : kb;  // (a lane without a second piece re-reads the first and does not use it)
    uint4 wv[FPW], wv2[FPW];
#pragma unroll
    for (int j = 0; j < FPW; ++j) wv[j] = load_weights<NT>(wrow[j] + kb);
#pragma unroll
    for (int j = 0; j < FPW; ++j) wv2[j] = load_weights<NT>(wrow[j] + kb2);
    const uint4 xv = *reinterpret_cast<const uint4*>(x + kb), xv2 = *reinterpret_cast<const uint4*>(x + kb2);
    add(wv, xv);
    if (two) add(wv2, xv2);
  }
#pragma unroll
  for (int j = 0; j < FPW; ++j) acc[j] = sum_lanes(acc[j]);
  if constexpr (KSPLIT) {  // the wavefronts' sums meet, in wavefront order
    if (lane < FPW) {
      float v = acc[0];
#pragma unroll
      for (int j = 1; j < FPW; ++j) v = lane == j ? acc[j] : v;
      red[wave][lane] = v;
    }
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int j = 0; j < FPW; ++j) {
      float v = red[0][j];
#pragma unroll
      for (int w = 1; w < GV_WAVES; ++w) v += red[w][j];
      acc[j] = v;
    }
  }
  if (lane < OUTF) {
    const int n = n0 + lane;
    float v = acc[0];
#pragma unroll
    for (int j = 1; j < OUTF; ++j) v = lane == j ? acc[j] : v;
    float u = acc[FPW - OUTF], b = 0.f;
    if (EPI == GV_SWIGLU) {
#pragma unroll
      for (int j = 1; j < OUTF; ++j) u = lane == j ? acc[FPW - OUTF + j] : u;
    } else if (bias) {
      b = lo16((uint32_t)bias[(eoff ? eoff[e] : (int64_t)e * N) + n]);
    }
    out[(size_t)row * N + n] = bf16_of(first_end<EPI>(v, u, b));
  }
}

// A step of ONE token with k >= 2 experts: the second product and the combine in one kernel.  A workgroup owns
// C1_FPW output features; two groups of four wavefronts take the k choices in turn (row = assign_to_row[j], its expert
// from the offsets table), split the contraction index, the sums meet in LDS in wavefront order, the result (+ bias)
// is rounded to bf16 and stored in yd as the separate product would store it, and out accumulates
// residual + sum_j w_j * yd[row_j] from those rounded values, in float32 and in the order of the combine kernel.
// One group (all choices one after the other) had half the loads in flight: 14.1 us for 64 experts of 2048 x 8192, k 2, 13.1 with two.
constexpr int C1_FPW = 8, C1_GROUPS = 2;

template <bool NT>
__global__ __launch_bounds__(C1_GROUPS * GV_WAVES * 64) void expert_gemv_combine1_kernel(
    const uint16_t* __restrict__ h, const uint16_t* __restrict__ w2, const uint16_t* __restrict__ bias,
    const int32_t* __restrict__ offsets, const int32_t* __restrict__ a2r, const float* __restrict__ topk_w,
    const uint16_t* residual, uint16_t* __restrict__ yd, uint16_t* out, const int64_t* __restrict__ eoff, int E, int N,
    int K, int k) {
  __shared__ int s_e[MOE_MAX_TOPK];  // expert of dispatched row r (T = 1: at most k rows)
  __shared__ float red[C1_GROUPS][GV_WAVES][C1_FPW];
  __shared__ float ys[MOE_MAX_TOPK][C1_FPW];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) % GV_WAVES);
  const int group = __builtin_amdgcn_readfirstlane(threadIdx.x / (GV_WAVES * 64)), gt = threadIdx.x % (GV_WAVES * 64);
  for (int e = threadIdx.x; e < E; e += C1_GROUPS * GV_WAVES * 64)
    for (int r = offsets[e]; r < offsets[e + 1] && r < MOE_MAX_TOPK; ++r) s_e[r] = e;
  __syncthreads();
  const int n0 = blockIdx.x * C1_FPW;
  float o = 0.f;  // (used by the first C1_FPW threads: output feature n0 + lane)
  if (threadIdx.x < C1_FPW && residual) o = lo16((uint32_t)residual[n0 + lane]);
  for (int j0 = 0; j0 < k; j0 += C1_GROUPS) {
    const int j = j0 + group, row = j < k ? a2r[j] : -1;
    if (row >= 0) {  // (else no choice, or a selection that is no expert: NaN logits; uniform per group)
      const int e = s_e[row];
      const uint16_t* wbase = w2 + (eoff ? eoff[e] : (int64_t)e * N * K) + (int64_t)n0 * K;
      const uint16_t* xrow = h + (int64_t)row * K;
      float acc[C1_FPW];
#pragma unroll
      for (int f = 0; f < C1_FPW; ++f) acc[f] = 0.f;
#pragma unroll 2
      for (int kb = gt * 8; kb < K; kb += GV_WAVES * 64 * 8) {
        uint4 wv[C1_FPW];
#pragma unroll
        for (int f = 0; f < C1_FPW; ++f) wv[f] = load_weights<NT>(wbase + (int64_t)f * K + kb);
        const uint4 xv = *reinterpret_cast<const uint4*>(xrow + kb);
        const Row8 x = unpack8(xv);
#pragma unroll
        for (int f = 0; f < C1_FPW; ++f) acc[f] = add8(acc[f], wv[f], x);
      }
      float mine = 0.f;  // lane f < C1_FPW: the wavefront's sum for output feature n0 + f
#pragma unroll
      for (int f = 0; f < C1_FPW; ++f) {
        const float v = sum_lanes(acc[f]);
        mine = lane == f ? v : mine;
      }
      if (lane < C1_FPW) red[group][wave][lane] = mine;
    }
    __syncthreads();
    if (row >= 0 && gt < C1_FPW) {
      float v = red[group][0][lane];
#pragma unroll
      for (int w = 1; w < GV_WAVES; ++w) v += red[group][w][lane];
      if (bias) v += lo16((uint32_t)bias[(eoff ? eoff[s_e[row]] : (int64_t)s_e[row] * N) + n0 + lane]);
      const uint16_t yb = bf16_of(v);
      yd[(size_t)row * N + n0 + lane] = yb;
      ys[j][lane] = lo16((uint32_t)yb);
    }
    __syncthreads();  // (red is free for the next choices)
  }
  if (threadIdx.x < C1_FPW) {
    for (int j = 0; j < k; ++j)
      if (a2r[j] >= 0) o = fmaf(topk_w[j], ys[j][lane], o);
    out[n0 + lane] = bf16_of(o);
  }
}

// Long rows and too few workgroups even so (`blocks` blocks of output features for `rows` rows): the wavefronts of a workgroup split
// the contraction index instead of the output features.
bool splits_contraction(int K, int blocks, int rows) { return K >= 4096 && (int64_t)blocks * rows < 512; }

template <int EPI, int ROWS, int FPW>
int32_t launch_shape(const moe_config* cfg, const uint16_t* act, const uint16_t* wa, const uint16_t* wb, const uint16_t* bias,
                     const int32_t* offsets, uint16_t* out, const int32_t* row_map, const float* gate_w, const uint16_t* residual,
                     const int32_t* a2r, const int64_t* eoff, int N, int K, bool gather, hipStream_t s) {
  constexpr int OUTF = EPI == GV_SWIGLU ? FPW / 2 : FPW;
  // About 256 KB of weights per workgroup, in whole blocks of output features, as long as that leaves about two
  // workgroups per CU (the experts with rows are at most k*T).
  const int A = cfg->k * cfg->T;
  int blocks = N / (GV_WAVES * OUTF);
  const bool ksplit = splits_contraction(K, blocks, A);
  if (ksplit) blocks *= GV_WAVES;
  int reps = ksplit ? 1 : (int)((256 * 1024) / ((int64_t)GV_WAVES * FPW * K * 2));
  reps = reps < 1 ? 1 : reps > 8 ? 8 : reps;
  while (reps > 1 && (blocks % reps || (int64_t)(blocks / reps) * A < 512)) --reps;
  const dim3 grid(blocks / reps, A), block(GV_WAVES * 64);
  const bool nt = weights_exceed_cache(cfg);
#define MOESYS_GEMV(G, S)                                                                                                  \
  hipLaunchKernelGGL((nt ? expert_gemv_kernel<EPI, G, ROWS, FPW, S, true> : expert_gemv_kernel<EPI, G, ROWS, FPW, S, false>), grid, block, 0, s, act, wa, wb, bias, offsets, out, row_map, \
                     gate_w, residual, a2r, eoff, cfg->T, cfg->E, N, K, reps)
  if (gather) { if (ksplit) MOESYS_GEMV(true, true); else MOESYS_GEMV(true, false); }
  else { if (ksplit) MOESYS_GEMV(false, true); else MOESYS_GEMV(false, false); }
#undef MOESYS_GEMV
  return check_hip(hipGetLastError(), "expert GEMV launch");
}

template <int EPI>
int32_t launch(const moe_config* cfg, const uint16_t* act, const uint16_t* wa, const uint16_t* wb, const uint16_t* bias,
               const int32_t* offsets, uint16_t* out, const int32_t* row_map, const float* gate_w, const uint16_t* residual,
               const int32_t* a2r, const int64_t* eoff, int N, int K, bool gather, hipStream_t s) {
  const int A = cfg->k * cfg->T;
  if (A == 0) return MOE_OK;
  if (A <= 8) return launch_shape<EPI, 8, 8>(cfg, act, wa, wb, bias, offsets, out, row_map, gate_w, residual, a2r, eoff, N, K, gather, s);
  return launch_shape<EPI, 16, 4>(cfg, act, wa, wb, bias, offsets, out, row_map, gate_w, residual, a2r, eoff, N, K, gather, s);
}

}  // namespace

// Whether the few-row path serves this product: so few assignments that no expert exceeds GV_MAX_ROWS rows,
// whole workgroups of output features, 16-byte chunks of the contraction index.
bool expert_gemv_applies(const moe_config* cfg, int N, int K) {
  const int64_t A = (int64_t)cfg->k * cfg->T;
  if (!tuning(MOE_TUNE_FEW_TOKEN_KERNELS) || cfg->dtype != MOE_BF16 || N % (GV_WAVES * 8) || K % 8) return false;
  // (with so few rows per expert the choice of the weight-streaming kernels does not depend on the activation)
  return A <= 8 || (A <= GV_MAX_ROWS && !expert_stream_applies(cfg, N, K, GV_BIAS));
}

// Second product + combine of a one-token step (k >= 2); see the kernel.  residual nullable; out may be residual.
bool expert_gemv_combine_one_token_applies(const moe_config* cfg) {
  return cfg->T == 1 && cfg->k >= 2 && expert_gemv_applies(cfg, cfg->d_model, cfg->d_ff);
}
int32_t launch_expert_gemv_combine_one_token(const moe_config* cfg, const void* h, const void* w2, const void* bias,
                                             const int32_t* offsets, const int32_t* a2r, const float* topk_w,
                                             const void* residual, void* yd, void* out, const int64_t* eoff, hipStream_t s) {
  if (!expert_gemv_combine_one_token_applies(cfg)) return fail(MOE_ERR_UNSUPPORTED, "expert GEMV: not a one-token step");
  hipLaunchKernelGGL(weights_exceed_cache(cfg) ? expert_gemv_combine1_kernel<true> : expert_gemv_combine1_kernel<false>, dim3(cfg->d_model / C1_FPW), dim3(C1_GROUPS * GV_WAVES * 64), 0, s, (const uint16_t*)h,
                     (const uint16_t*)w2, (const uint16_t*)bias, offsets, a2r, topk_w, (const uint16_t*)residual, (uint16_t*)yd,
                     (uint16_t*)out, eoff, cfg->E, cfg->d_model, cfg->d_ff, cfg->k);
  return check_hip(hipGetLastError(), "expert GEMV launch");
}

// Ranking + first product of a one-token step, from the partial logits of launch_gate_parts_one_token (at most 16 slices).
bool expert_gemv_ranked_applies(const moe_config* cfg) {
  return expert_gemv_combine_one_token_applies(cfg) && cfg->E <= 64 && expert_gemv_applies(cfg, cfg->d_ff, cfg->d_model);
}
int32_t launch_rank_one_token(const moe_config* cfg, const double* part, int slices, const float* b_router, int32_t* topk_idx, float* topk_w,
                              int32_t* counts, int32_t* offsets, int32_t* a2r, int32_t* r2a, int32_t* clear8, hipStream_t s) {
  if (!expert_gemv_ranked_applies(cfg) || slices < 1 || slices > RANKED_SLICES) return fail(MOE_ERR_UNSUPPORTED, "expert GEMV: not a ranked one-token step");
  hipLaunchKernelGGL(rank_one_token_kernel, dim3(1), dim3(GV_WAVES * 64), 0, s, part, slices, b_router, cfg->renormalize, topk_idx, topk_w,
                     counts, offsets, a2r, r2a, clear8, cfg->E, cfg->k);
  return check_hip(hipGetLastError(), "gate launch");
}
int32_t launch_expert_gemv_ranked(const moe_config* cfg, const void* x, const double* part, int slices, const float* b_router, const void* wa,
                                  const void* wb, const void* bias, void* h, const int64_t* eoff, int32_t* topk_idx, float* topk_w,
                                  int32_t* counts, int32_t* offsets, int32_t* a2r, int32_t* r2a, int32_t* clear8, hipStream_t s) {
  if (!expert_gemv_ranked_applies(cfg) || slices < 1 || slices > RANKED_SLICES) return fail(MOE_ERR_UNSUPPORTED, "expert GEMV: not a ranked one-token step");
  const int N = cfg->d_ff;
  const bool sw = cfg->act == MOE_ACT_SWIGLU, nt = weights_exceed_cache(cfg);
  const int per8 = GV_WAVES * (sw ? 4 : 8);  // output features per workgroup with eight weight rows per wavefront
  const bool ksplit = splits_contraction(cfg->d_model, N / per8, cfg->k);
  const int of8 = ksplit ? per8 / GV_WAVES : per8;
  const bool eight = (int64_t)(N / of8) * cfg->k >= 512;  // about two workgroups per CU, else half the rows
  const dim3 grid(N / (eight ? of8 : of8 / 2), cfg->k), block(GV_WAVES * 64);
#define MOESYS_RANKED(EP, F)                                                                                                      \
  hipLaunchKernelGGL((ksplit ? (nt ? expert_gemv_ranked_kernel<EP, F, true, true> : expert_gemv_ranked_kernel<EP, F, false, true>)  \
                             : (nt ? expert_gemv_ranked_kernel<EP, F, true, false> : expert_gemv_ranked_kernel<EP, F, false, false>)), \
                     grid, block, 0, s,                                                                                           \
                     (const uint16_t*)x, part, slices, b_router, cfg->renormalize, (const uint16_t*)wa, (const uint16_t*)wb,       \
                     (const uint16_t*)bias, (uint16_t*)h, eoff, topk_idx, topk_w, counts, offsets, a2r, r2a, clear8, cfg->E, N,    \
                     cfg->d_model, cfg->k)
  if (sw) { if (eight) MOESYS_RANKED(GV_SWIGLU, 8); else MOESYS_RANKED(GV_SWIGLU, 4); }
  else { if (eight) MOESYS_RANKED(GV_GELU, 8); else MOESYS_RANKED(GV_GELU, 4); }
#undef MOESYS_RANKED
  return check_hip(hipGetLastError(), "expert GEMV launch");
}

// epi: 0 GELU (+bias), 1 SwiGLU (wa = gate, wb = up), 2 plain (+bias), 3 combine for k = 1 (row_map = row_to_assign,
// gate_w, residual; a2r or NULL: fill_rowless_tokens).  row_map with epi 0/1: gather the rows from x[T, K].  eoff: per-expert element offsets or NULL.
int32_t launch_expert_gemv_bf16(int epi, const moe_config* cfg, const void* act, const void* wa, const void* wb, const void* bias,
                                const int32_t* offsets, void* out, const int32_t* row_map, const float* gate_w,
                                const void* residual, const int32_t* a2r, const int64_t* eoff, int N, int K, hipStream_t s) {
  if (!expert_gemv_applies(cfg, N, K)) return fail(MOE_ERR_UNSUPPORTED, "expert GEMV: shape outside the few-row path");
  const uint16_t *a = (const uint16_t*)act, *w0 = (const uint16_t*)wa, *w1 = (const uint16_t*)wb, *b = (const uint16_t*)bias;
  const uint16_t* res = (const uint16_t*)residual;
  switch (epi) {
    case GV_GELU: return launch<GV_GELU>(cfg, a, w0, w1, b, offsets, (uint16_t*)out, row_map, gate_w, res, a2r, eoff, N, K, row_map != nullptr, s);
    case GV_SWIGLU: return launch<GV_SWIGLU>(cfg, a, w0, w1, nullptr, offsets, (uint16_t*)out, row_map, gate_w, res, a2r, eoff, N, K, row_map != nullptr, s);
    case GV_BIAS: return launch<GV_BIAS>(cfg, a, w0, w1, b, offsets, (uint16_t*)out, nullptr, gate_w, res, a2r, eoff, N, K, false, s);
    case GV_COMBINE:
      if (!row_map || !gate_w || cfg->k != 1) return fail(MOE_ERR_INVALID_ARG, "expert GEMV: combine epilogue needs k = 1, row map and gate weights");
      return launch<GV_COMBINE>(cfg, a, w0, w1, b, offsets, (uint16_t*)out, row_map, gate_w, res, a2r, eoff, N, K, false, s);
  }
  return fail(MOE_ERR_INVALID_ARG, "expert GEMV: unknown epilogue");
}

}  // namespace moesys
