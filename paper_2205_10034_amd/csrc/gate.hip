// Top-k softmax gate (GShard top-2 / top-1 gating, Section 5.2; softmax in fp32, Section 5.2).
//
// Fast path (bf16 activations, E <= 64; the rules that choose are at launch_gate), HBM-bound: the logits are a skinny GEMM on the MFMA units.
// Activations are bfloat16 already; every float32 router weight is split into three bfloat16 pieces
// (w = hi + mid + lo exactly), so every product is exact in float32 and the only rounding is the
// accumulation: float32 inside a 64-wide K chunk (24 roundings at most), float64 across chunks and
// across the four wavefronts that share the K range.  The logits therefore carry an error of about
// 1e-7.  Ranking needs more: it must equal the ranking of the exactly computed logits.  Any token whose
// k+1 leading logits have two neighbours closer than GATE_MARGIN_REL times its largest |logit| is recomputed by the whole workgroup
// with float64 accumulation of the (exact) products and ranked on those values.
//
// Exact path (float32 activations, E > 64, many tokens on more than 16 experts by gate_f64_pays, and inside a layer steps of up to
// 256 tokens, in slices of the contraction index): the products of two float32 / bfloat16 values are exact in float64, and
// v_mfma_f64_16x16x4_f64 accumulates them there, so only the summation rounds, at 2^-53 relative, and nothing has to be
// recomputed; see gate_f64_kernel and gate_rank_kernel.
#include "gate_rank.h"
#include "moesys_internal.h"
#include "routing_tables.h"
#include "wave_util.h"

namespace moesys {
namespace {

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ __forceinline__ double shfl_xor_f64(double v, int m) {
  int lo = __double2loint(v), hi = __double2hiint(v);
  lo = __shfl_xor(lo, m, 64);
  hi = __shfl_xor(hi, m, 64);
  return __hiloint2double(hi, lo);
}

// One wavefront ranks one token from its float64 logits z[0..E): softmax in float32 (row maximum subtracted),
// k rounds of arg-max on the float64 logits (ties -> lower expert index), weights p or p / sum of the selected.
// Returns the j-th selected expert in lane j < k (0 in the other lanes).
__device__ __forceinline__ int rank_token(const double* z, int lane, int E, int k, int renorm, int t,
                                          int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                          float* __restrict__ probs) {
  // each lane owns experts lane, lane+64, ...
  double zd[4];
  float zf[4];
  float mx = -INFINITY;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int e = lane + 64 * s;
    zd[s] = e < E ? z[e] : -INFINITY;
    zf[s] = (float)zd[s];
    mx = fmaxf(mx, zf[s]);
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) mx = fmaxf(mx, __shfl_xor(mx, m, 64));
  float ex[4], sum = 0.f;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    ex[s] = (lane + 64 * s) < E ? expf(zf[s] - mx) : 0.f;
    sum += ex[s];
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) sum += __shfl_xor(sum, m, 64);
  float p[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    p[s] = ex[s] / sum;
    if (probs && (lane + 64 * s) < E) probs[(size_t)t * E + lane + 64 * s] = p[s];
  }
  // k rounds of arg-max on the float64 logits; ties -> lower expert index
  float wsel = 0.f, wsum = 0.f;  // lane j keeps the j-th selection
  int isel = 0;
  for (int j = 0; j < k; ++j) {
    double bz = -INFINITY;
    int be = 0x7fffffff;
    float bp = 0.f;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int e = lane + 64 * s;
      if (e < E && (zd[s] > bz || (zd[s] == bz && e < be))) { bz = zd[s]; be = e; bp = p[s]; }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
      double oz = shfl_xor_f64(bz, m);
      int oe = __shfl_xor(be, m, 64);
      float op = __shfl_xor(bp, m, 64);
      if (oz > bz || (oz == bz && oe < be)) { bz = oz; be = oe; bp = op; }
    }
    // retire the winner (all lanes agree on be): as NaN, which no comparison picks again, also where what is left is -inf
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (lane + 64 * s == be) zd[s] = NAN;
    if (lane == j) { isel = be; wsel = bp; }
    wsum += bp;
  }
  if (lane < k) {
    topk_idx[(size_t)t * k + lane] = isel;
    topk_w[(size_t)t * k + lane] = renorm ? wsel / wsum : wsel;
  }
  return isel;
}

// Few tokens (T <= FEW_MAX_T; E = 4, 8, 16, 32 or 64): one workgroup per token, so that the whole router matrix
// is not read through one compute unit's handful of wavefronts, with loads that are contiguous across the
// wavefront: a router row is E/4 chunks of four floats; lane (r, c) of a wavefront reads chunk c of the r-th of
// the 64 / (E/4) rows that one wave-wide load covers, and accumulates those four logits in float64 (exact
// products, see above) over its share of the rows.  The sums meet across the row groups of a wavefront by a
// butterfly, across the wavefronts in wavefront order, and wavefront 0 ranks the token.
constexpr int FEW_MAX_T = 16;
constexpr int FEW_WAVES = 16;  // (all the loads of a token are in flight in two batches at d_model = 2048)
constexpr int FEW_THREADS = FEW_WAVES * 64;

template <typename XT>
__global__ __launch_bounds__(FEW_THREADS) void gate_few_kernel(
    const XT* __restrict__ x, const float* __restrict__ wr, const float* __restrict__ br, int T, int d, int E, int k,
    int renorm, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w, float* __restrict__ probs,
    int32_t* __restrict__ counts, int32_t* __restrict__ offsets, int32_t* __restrict__ a2r, int32_t* __restrict__ r2a,
    int32_t* __restrict__ clear8) {
  __shared__ double part[FEW_WAVES][64];
  __shared__ double zrow[64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t = blockIdx.x;
  const int cpr = E >> 2, rpi = 64 / cpr;  // chunks per row, rows per wave-wide load
  const int r = lane / cpr, c = lane % cpr;
  const XT* xt = x + (size_t)t * d;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
#pragma unroll 16
  for (int row = wave * rpi + r; row < d; row += FEW_WAVES * rpi) {
    const float4 w4 = *reinterpret_cast<const float4*>(wr + (size_t)row * E + 4 * c);
    float xv;
    if constexpr (sizeof(XT) == 2) xv = bf16_to_f32(xt[row]);
    else xv = xt[row];
    const double xd = (double)xv;
    a0 = fma(xd, (double)w4.x, a0);
    a1 = fma(xd, (double)w4.y, a1);
    a2 = fma(xd, (double)w4.z, a2);
    a3 = fma(xd, (double)w4.w, a3);
  }
  for (int m = cpr; m < 64; m <<= 1) {  // lanes with the same chunk sit cpr apart
    a0 += shfl_xor_f64(a0, m);
    a1 += shfl_xor_f64(a1, m);
    a2 += shfl_xor_f64(a2, m);
    a3 += shfl_xor_f64(a3, m);
  }
  if (lane < cpr) {
    part[wave][4 * c] = a0; part[wave][4 * c + 1] = a1; part[wave][4 * c + 2] = a2; part[wave][4 * c + 3] = a3;
  }
  __syncthreads();
  if ((int)threadIdx.x < E) {
    double zsum = 0.0;
#pragma unroll
    for (int w = 0; w < FEW_WAVES; ++w) zsum += part[w][threadIdx.x];
    zrow[threadIdx.x] = zsum + (br ? (double)br[threadIdx.x] : 0.0);
  }
  __syncthreads();
  if (wave != 0) return;
  const int sel = rank_token(zrow, lane, E, k, renorm, t, topk_idx, topk_w, probs);
  // A step of ONE token (counts != NULL; T == 1): its dispatch tables follow from the selection at once.  The k
  // experts are distinct and get one row each (the capacity is at least one; only a selection that is no expert is
  // dropped); rows are ordered by expert; assignment j (= j*T + t with T = 1) is the j-th choice.
  if (counts) {
    const int mine = valid_expert(sel, E);
    unsigned long long chosen = 0;  // bit e: expert e selected (E <= 64)
    for (int j = 0; j < k; ++j) {
      const int e = __shfl(mine, j, 64);
      if (e >= 0) chosen |= 1ull << e;
    }
    if (lane < E) {
      counts[lane] = (int)((chosen >> lane) & 1ull);
      offsets[lane] = __popcll(chosen & ((1ull << lane) - 1ull));
    }
    if (lane == 0) offsets[E] = __popcll(chosen);
    if (lane < k) {
      const int row = mine >= 0 ? __popcll(chosen & ((1ull << mine) - 1ull)) : -1;
      a2r[lane] = row;
      if (row >= 0) r2a[row] = lane;
    }
    if (clear8 && lane < 8) clear8[lane] = 0;
  }
}

// the shapes the kernel above is written for
bool gate_few_applies(const moe_config* cfg, const float* w_router) {
  const int E = cfg->E;
  return tuning(MOE_TUNE_FEW_TOKEN_KERNELS) != 0 && cfg->T <= FEW_MAX_T && (E == 4 || E == 8 || E == 16 || E == 32 || E == 64) &&
         (reinterpret_cast<uintptr_t>(w_router) & 15) == 0;
}

template <typename XT>
int32_t launch_few(const moe_config* cfg, const void* x, const float* w_router, const float* b_router, int32_t* topk_idx,
                   float* topk_w, float* probs, hipStream_t s, int32_t* counts = nullptr, int32_t* offsets = nullptr,
                   int32_t* a2r = nullptr, int32_t* r2a = nullptr, int32_t* clear8 = nullptr) {
  hipLaunchKernelGGL(gate_few_kernel<XT>, dim3(cfg->T), dim3(FEW_THREADS), 0, s, (const XT*)x, w_router, b_router, cfg->T,
                     cfg->d_model, cfg->E, cfg->k, cfg->renormalize, topk_idx, topk_w, probs, counts, offsets, a2r, r2a, clear8);
  return check_hip(hipGetLastError(), "gate launch");
}

// ------------------------------------------------------------------------------------------------
// Fast path.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int FT_TOK = 16;           // tokens per workgroup (one 16-token MFMA tile)
constexpr int FT_KC = 64;            // K chunk: two 16x16x32 MFMA steps
constexpr int FT_ROW = (FT_KC + 8) * 2;  // LDS row of one expert's chunk, padded to 144 B (conflict-free reads)
// neighbours among the k+1 leading logits closer than this times the token's largest |logit| -> exact recompute
// (the accumulation error scales with the data; for inputs of unit variance this is about 1e-4)
constexpr float GATE_MARGIN_REL = 1.0f / 32768.0f;

__device__ __forceinline__ uint32_t bf16_bits_rne(float f) { return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)f); }

// ------------------------------------------------------------------------------------------------
// Exact path: 16 tokens per workgroup, every expert; the wavefronts split the contraction index and their float64 sums
// meet in LDS in wavefront order.
//
// One v_mfma_f64_16x16x4_f64 takes 16 experts x 16 tokens x 4 values: lane l supplies router row k = l / 16 for expert
// q = l mod 16 and the activation of token l mod 16.  A dot product does not care about the order of its terms, so lane
// group g = l / 16 takes a run of KPL consecutive values of a chunk of 4 KPL (one load of the token's row for KPL MFMA
// steps), and expert q of an MFMA is any expert as long as the result is read back the same way: with EV experts per
// lane, one load of EV consecutive router weights feeds the EV MFMAs of a group of 16 EV experts.  Operands are
// converted in registers; the loads of the next chunk are in flight while a chunk is multiplied.
// Bound by the latency of that chain for few tokens and by the float64 matrix rate for many: the vector-ALU kernel that
// was here re-read its token rows once per 16 experts and its router weights uncoalesced and element by element.  Measured
// on MI355X (us, before -> now): bf16, 128 experts: 3001 x 1600 499 -> 45, 16384 x 4096 4612 -> 329 (52 TFLOP/s of the
// 78.6 that float64 MFMAs can do); 256 experts, 2048 x 2048 1068 -> 100; float32, 16 experts, 2048 x 1024 45 -> 7.4;
// 64 experts, 4096 x 1024 158 -> 17.
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int F64_TOK = 16;

// values of the contraction index per lane and chunk (two chunks have to fit the registers beside the sums)
template <typename XT, int EV, int NG, bool VEC>
constexpr int f64_values() { return sizeof(XT) == 4 || NG > 2 || (EV == 4 && (NG == 1 || !VEC)) ? 4 : 8; }

// PART: workgroup (x, y) multiplies only the chunks [y chunks_per, (y + 1) chunks_per) and stores the sums of its 16 tokens, the
// partial logits part[y][token][expert], for gate_rank_kernel or for a product that ranks by itself.
template <typename XT, int EV, int NG, bool VEC, int NW, bool PART = false>
__global__ __launch_bounds__(NW * 64) void gate_f64_kernel(const XT* __restrict__ x, const float* __restrict__ wr,
                                                           const float* __restrict__ br, int T, int d, int E, int k, int renorm,
                                                           int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                                           float* __restrict__ probs, int chunks_per, double* __restrict__ part) {
  constexpr int KPL = f64_values<XT, EV, NG, VEC>();
  constexpr int KC = 4 * KPL, EP = 16 * EV * NG, NPL = EP / 8;
  extern __shared__ double part64[];  // [NW][EP][F64_TOK]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane & 15, g = lane >> 4;
  const int t0 = blockIdx.x * F64_TOK;
  const XT* xrow = x + (size_t)min(t0 + q, T - 1) * d + g * KPL;  // (tail tokens redo the last row and are not stored)

  int e0[NG];  // first of this lane's EV experts in group n, moved into range (what a row past the last expert yields is not read)
#pragma unroll
  for (int n = 0; n < NG; ++n) e0[n] = (n * 16 + q) * EV < E ? (n * 16 + q) * EV : 0;
  struct Chunk { float w[KPL][NG][EV]; float xv[KPL]; };
  auto load = [&](int c, Chunk& b) {
    const XT* xp = xrow + (size_t)c * KC;
    if constexpr (sizeof(XT) == 4) {
      const float4 v = *reinterpret_cast<const float4*>(xp);
      b.xv[0] = v.x; b.xv[1] = v.y; b.xv[2] = v.z; b.xv[3] = v.w;
    } else {
      uint32_t u[KPL / 2];
      if constexpr (KPL == 8) {
        const uint4 v = *reinterpret_cast<const uint4*>(xp);
        u[0] = v.x; u[1] = v.y; u[2] = v.z; u[3] = v.w;
      } else {
        const uint2 v = *reinterpret_cast<const uint2*>(xp);
        u[0] = v.x; u[1] = v.y;
      }
#pragma unroll
      for (int i = 0; i < KPL / 2; ++i) {
        b.xv[2 * i] = __uint_as_float(u[i] << 16);
        b.xv[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
      }
    }
#pragma unroll
    for (int s = 0; s < KPL; ++s) {
      const float* row = wr + (size_t)(c * KC + g * KPL + s) * E;
#pragma unroll
      for (int n = 0; n < NG; ++n) {
        if constexpr (VEC && EV == 4) {
          const float4 v = *reinterpret_cast<const float4*>(row + e0[n]);
          b.w[s][n][0] = v.x; b.w[s][n][1] = v.y; b.w[s][n][2] = v.z; b.w[s][n][3] = v.w;
        } else if constexpr (VEC && EV == 2) {
          const float2 v = *reinterpret_cast<const float2*>(row + e0[n]);
          b.w[s][n][0] = v.x; b.w[s][n][1] = v.y;
        } else {
#pragma unroll
          for (int j = 0; j < EV; ++j) b.w[s][n][j] = row[min(e0[n] + j, E - 1)];
        }
      }
    }
  };
  f64x4 acc[NG][EV];
#pragma unroll
  for (int n = 0; n < NG; ++n)
#pragma unroll
    for (int j = 0; j < EV; ++j) acc[n][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  auto multiply = [&](const Chunk& b) {
#pragma unroll
    for (int s = 0; s < KPL; ++s) {
      const double xd = (double)b.xv[s];
#pragma unroll
      for (int n = 0; n < NG; ++n)
#pragma unroll
        for (int j = 0; j < EV; ++j) acc[n][j] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)b.w[s][n][j], xd, acc[n][j], 0, 0, 0);
    }
  };
  const int first = PART ? (int)blockIdx.y * chunks_per + wave : wave;
  const int n_chunks = PART ? min(d / KC, ((int)blockIdx.y + 1) * chunks_per) : d / KC;  // (the end; d is a multiple of 64)
  if (first < n_chunks) {
    Chunk b[2];
    load(first, b[0]);
    int c = first;
    for (; c + NW < n_chunks; c += 2 * NW) {
      load(c + NW, b[1]);
      multiply(b[0]);
      load(min(c + 2 * NW, n_chunks - 1), b[0]);
      multiply(b[1]);
    }
    if (c < n_chunks) multiply(b[0]);
  }
  // accumulator register i of lane (q, g): row 4 i + g of the MFMA, token q
#pragma unroll
  for (int n = 0; n < NG; ++n)
#pragma unroll
    for (int j = 0; j < EV; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        part64[((size_t)wave * EP + (n * 16 + 4 * i + g) * EV + j) * F64_TOK + q] = acc[n][j][i];
  lds_barrier();
  if constexpr (PART) {
    double* dst = part + ((size_t)blockIdx.y * T + t0) * E;
    for (int i = tid; i < EP * F64_TOK; i += NW * 64) {
      const int e = i / F64_TOK, tok = i % F64_TOK;
      if (e >= E || t0 + tok >= T) continue;
      double v = part64[i];
#pragma unroll
      for (int w = 1; w < NW; ++w) v += part64[(size_t)w * EP * F64_TOK + i];
      dst[tok * E + e] = v;
    }
    return;
  }
  for (int i = tid; i < EP * F64_TOK; i += NW * 64) {  // (a sum's first term is its own place: nobody else touches it)
    double v = part64[i];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += part64[(size_t)w * EP * F64_TOK + i];
    const int e = i / F64_TOK;
    part64[i] = v + (br && e < E ? (double)br[e] : 0.0);
  }
  lds_barrier();
  for (int i = tid; i < F64_TOK * 8; i += NW * 64) {
    const int tok = i >> 3, sub = i & 7, t = t0 + tok;
    double z[NPL];
#pragma unroll
    for (int m = 0; m < NPL; ++m) z[m] = sub + 8 * m < E ? part64[(sub + 8 * m) * F64_TOK + tok] : -INFINITY;
    if (t < T)
      finalize_group<NPL, false>(z, sub, E, k, renorm, 0.f, topk_idx + (size_t)t * k, topk_w + (size_t)t * k,
                                 probs ? probs + (size_t)t * E : nullptr);
  }
}

template <typename XT, int EV, int NG, int NW>
int32_t launch_f64_shape(const moe_config* cfg, const void* x, const float* w_router, const float* b_router, int32_t* topk_idx,
                         float* topk_w, float* probs, hipStream_t s) {
  constexpr size_t shmem = (size_t)NW * 16 * EV * NG * F64_TOK * sizeof(double);
  static_assert(shmem <= 128 * 1024, "the partial sums do not fit the LDS");
  const bool vec = cfg->E % EV == 0 && ((uintptr_t)w_router & (4 * EV - 1)) == 0;
  auto kern = vec ? gate_f64_kernel<XT, EV, NG, true, NW> : gate_f64_kernel<XT, EV, NG, false, NW>;
  if (shmem > 65536) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
    if (e != hipSuccess) return check_hip(e, "hipFuncSetAttribute(gate LDS)");
  }
  hipLaunchKernelGGL(kern, dim3((cfg->T + F64_TOK - 1) / F64_TOK), dim3(NW * 64), shmem, s, (const XT*)x, w_router, b_router, cfg->T,
                     cfg->d_model, cfg->E, cfg->k, cfg->renormalize, topk_idx, topk_w, probs, 0, (double*)nullptr);
  return check_hip(hipGetLastError(), "gate launch");
}

// wavefronts: as many as keep the partial sums within 128 KB of LDS
template <typename XT>
int32_t launch_f64(const moe_config* cfg, const void* x, const float* w_router, const float* b_router, int32_t* topk_idx,
                   float* topk_w, float* probs, hipStream_t s) {
  if (cfg->E <= 16) return launch_f64_shape<XT, 1, 1, 16>(cfg, x, w_router, b_router, topk_idx, topk_w, probs, s);
  if (cfg->E <= 32) return launch_f64_shape<XT, 2, 1, 16>(cfg, x, w_router, b_router, topk_idx, topk_w, probs, s);
  if (cfg->E <= 64) return launch_f64_shape<XT, 4, 1, 16>(cfg, x, w_router, b_router, topk_idx, topk_w, probs, s);
  if (cfg->E <= 128) return launch_f64_shape<XT, 4, 2, 8>(cfg, x, w_router, b_router, topk_idx, topk_w, probs, s);
  return launch_f64_shape<XT, 4, 4, 4>(cfg, x, w_router, b_router, topk_idx, topk_w, probs, s);
}

// ------------------------------------------------------------------------------------------------
// A step of a few hundred tokens at most: 16 tokens per workgroup leave most compute units without work and each with the whole
// router to read, and the dispatch tables of so few assignments cost a launch of their own.  So the contraction index is cut into
// slices as well (gate_f64_kernel with PART: float64 sums, nothing to recompute), and one workgroup adds the slices in order,
// ranks every token in a group of eight lanes and writes the dispatch tables.  Bound by the latency of two launches.
// Measured on MI355X inside layers whose weights drive everything else out of the caches (us, a workgroup per 16 tokens + dispatch
// kernel / slices + this one): 96 tokens, d 4096, 8 experts 17.4 + 5.1 / 5.0 + 7.7; 96, d 2048, 64 23.9 + 4.9 / 7.5 + 11.3; 8, d 2048, 64
// (32 slices on the vector ALU and a ranking wavefront per token before) 9.4 + 7.5 / 5.0 + 7.4; whole layers: 32 tokens, d 2048, 128
// experts 191 / 162, 255, d 4096, 32 154 / 141, 3, d 1152, 24 43.4 / 38.3.  More than 96 tokens and short rows lose: 200, d 1024, 32
// experts and 256, d 1024, 8 to 16 by 1 to 2 us; 128 to 255 at d 1536 gain 2 to 3.
constexpr int GR_THREADS = ONE_WAVES * 64, GR_MAX_T = 256, GR_LOGITS = 8192;
// slices that a thread adds for each of its logits_per_thread logits: all of its loads are in flight together
constexpr int gr_slices(int logits_per_thread) { return logits_per_thread <= 4 ? 16 / logits_per_thread : 4; }
constexpr int gr_logits_per_thread(int logits) { return logits <= GR_THREADS ? 1 : logits <= 2 * GR_THREADS ? 2 : logits <= 4 * GR_THREADS ? 4 : 8; }
// WAVE_ORDER: steps whose gate alone would be gate_few_kernel get that kernel's weights, bit for bit, and so do their gradients.
template <int NPL, bool WAVE_ORDER>
__global__ __launch_bounds__(GR_THREADS) void gate_rank_kernel(const double* __restrict__ part, const float* __restrict__ br, int T, int E,
                                                               int k, int C, int renorm, int slices, int32_t* __restrict__ topk_idx,
                                                               float* __restrict__ topk_w, int32_t* __restrict__ counts,
                                                               int32_t* __restrict__ offsets, int32_t* __restrict__ a2r,
                                                               int32_t* __restrict__ r2a, int32_t* __restrict__ clear8) {
  // logits [token][E + 8] (the pad spreads the groups' reads over the banks), then the tables
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_rank[];
  __shared__ int sel[GR_THREADS];  // [T][k]
  double* zs = reinterpret_cast<double*>(smem_rank);
  const int tid = threadIdx.x, n = T * E;
  if (clear8 && tid < 8) clear8[tid] = 0;
  auto add_slices = [&](auto lpt) {
    constexpr int LPT = decltype(lpt)::value, S = gr_slices(LPT);
    double v[LPT][S];
#pragma unroll
    for (int q = 0; q < S; ++q) {
      const double* p = part + (size_t)min(q, slices - 1) * n;  // (uniform)
#pragma unroll
      for (int l = 0; l < LPT; ++l) v[l][q] = p[(unsigned)min(l * GR_THREADS + tid, n - 1)];
    }
#pragma unroll
    for (int l = 0; l < LPT; ++l) {
      const int i = l * GR_THREADS + tid;
      // i / E: at least 0.5 / E away from a whole number, which is 200 times what these float32 operations can be off
      const int t = (int)(((float)i + 0.5f) * __builtin_amdgcn_rcpf((float)E));
      double z = v[l][0];
#pragma unroll
      for (int q = 1; q < S; ++q) z += q < slices ? v[l][q] : 0.0;
      if (i < n) zs[i + 8 * t] = z + (br ? (double)br[i - t * E] : 0.0);
    }
  };
  switch (gr_logits_per_thread(n)) {
    case 1: add_slices(std::integral_constant<int, 1>{}); break;
    case 2: add_slices(std::integral_constant<int, 2>{}); break;
    case 4: add_slices(std::integral_constant<int, 4>{}); break;
    default: add_slices(std::integral_constant<int, 8>{});
  }
  __syncthreads();
  const int sub = tid & 7;
  for (int t = tid >> 3; t < T; t += GR_THREADS / 8) {  // (uniform per group)
    double z[NPL];
#pragma unroll
    for (int i = 0; i < NPL; ++i) z[i] = sub + 8 * i < E ? zs[t * (E + 8) + sub + 8 * i] : -INFINITY;
    finalize_group<NPL, false, WAVE_ORDER>(z, sub, E, k, renorm, 0.f, sel + t * k, topk_w + (size_t)t * k, nullptr);
  }
  __syncthreads();
  const int A = T * k, j = tid / T, t = tid - j * T;  // assignment j T + t
  if (tid < A) topk_idx[tid] = sel[tid];
  const int e_of[1] = {tid < A ? valid_expert(sel[t * k + j], E) : -1};
  write_tables<1>(e_of, A, E, C, *reinterpret_cast<OneTables*>(smem_rank), counts, offsets, a2r, r2a);
}

// The slices of the kernel above: as many as its threads add and the scratch holds; no slice gives a wavefront less than one chunk.
struct GateSlices { int slices, chunks_per, waves, logits; };
GateSlices plan_gate_slices(const moe_config* cfg, const float* w_router, size_t scratch_bytes) {
  const int T = cfg->T, E = cfg->E, ev = E <= 16 ? 1 : E <= 32 ? 2 : 4;
  GateSlices p = {0, 0, E <= 128 ? 8 : 4, T * E};
  const bool vec = E % ev == 0 && ((uintptr_t)w_router & (4 * ev - 1)) == 0;
  const int kc = 4 * (E <= 32 ? f64_values<uint16_t, 1, 1, true>() : E <= 64 || E > 128 || !vec ? 4 : f64_values<uint16_t, 4, 2, true>());
  int64_t most = gr_slices(gr_logits_per_thread(p.logits));
  const int64_t room = (int64_t)(scratch_bytes / ((size_t)p.logits * sizeof(double)));
  if (room < most) most = room;
  if (most < 1) return p;
  const int chunks = cfg->d_model / kc;
  p.chunks_per = (int)((chunks + most - 1) / most);
  if (p.chunks_per < p.waves) p.chunks_per = p.waves;
  p.slices = (chunks + p.chunks_per - 1) / p.chunks_per;
  return p;
}

template <int EV, int NG, int NW>
int32_t launch_gate_parts_shape(const moe_config* cfg, const GateSlices& p, const void* x, const float* w_router, double* part, hipStream_t s) {
  constexpr size_t shmem = (size_t)NW * 16 * EV * NG * F64_TOK * sizeof(double);
  const bool vec = cfg->E % EV == 0 && ((uintptr_t)w_router & (4 * EV - 1)) == 0;
  auto kern = vec ? gate_f64_kernel<uint16_t, EV, NG, true, NW, true> : gate_f64_kernel<uint16_t, EV, NG, false, NW, true>;
  if (shmem > 65536) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
    if (e != hipSuccess) return check_hip(e, "hipFuncSetAttribute(gate LDS)");
  }
  hipLaunchKernelGGL(kern, dim3((cfg->T + F64_TOK - 1) / F64_TOK, p.slices), dim3(NW * 64), shmem, s, (const uint16_t*)x, w_router,
                     (const float*)nullptr, cfg->T, cfg->d_model, cfg->E, cfg->k, cfg->renormalize, (int32_t*)nullptr, (float*)nullptr,
                     (float*)nullptr, p.chunks_per, part);
  return check_hip(hipGetLastError(), "gate launch");
}
int32_t launch_gate_parts(const moe_config* cfg, const GateSlices& p, const void* x, const float* w_router, double* part, hipStream_t s) {
  if (cfg->E <= 16) return launch_gate_parts_shape<1, 1, 8>(cfg, p, x, w_router, part, s);
  if (cfg->E <= 32) return launch_gate_parts_shape<2, 1, 8>(cfg, p, x, w_router, part, s);
  if (cfg->E <= 64) return launch_gate_parts_shape<4, 1, 8>(cfg, p, x, w_router, part, s);
  if (cfg->E <= 128) return launch_gate_parts_shape<4, 2, 8>(cfg, p, x, w_router, part, s);
  return launch_gate_parts_shape<4, 4, 4>(cfg, p, x, w_router, part, s);
}

// EB = number of 16-expert blocks (E <= 16*EB).  One workgroup = 16 tokens (one MFMA token tile); its NWV
// wavefronts split the K range chunk by chunk and meet once, to add their partial logits.  A wavefront
// works through a chunk one expert block at a time, re-using one staging area of 16 experts (its LDS
// operations execute in order), so that eight wavefronts fit where the router is wide: with 64 experts a
// wavefront's chain of split, stage and multiply is four times as long as with 16, and the kernel's time
// is the length of that chain.  VEC: the router weights can be read four experts at a time (E a multiple
// of 4, 16-byte aligned base).
template <int EB>
constexpr int gate_waves() { return EB == 1 ? 4 : 8; }

// TT = 16-token tiles per workgroup.  The split of the router into its three pieces is the larger part of a
// workgroup's work and does not depend on the tokens: two tiles share it (and the 64 KB of router a workgroup reads
// per 16 experts), which is worth it once there are enough tokens to keep every CU busy with half as many workgroups.
template <int EB, bool VEC, int TT>
__global__ __launch_bounds__(gate_waves<EB>() * 64) void gate_mfma_kernel(const uint16_t* __restrict__ x, const float* __restrict__ wr,
                                                        const float* __restrict__ br, int T, int d, int E, int k,
                                                        int renorm, int32_t* __restrict__ topk_idx,
                                                        float* __restrict__ topk_w, float* __restrict__ probs) {
  constexpr int EP = EB * 16;
  constexpr int NPL = EP / 8;                    // logits per lane in the 8-lane finalisation groups
  constexpr int NWV = gate_waves<EB>();
  constexpr int W_WAVE_BYTES = 3 * 16 * FT_ROW;  // one wavefront's hi/mid/lo pieces of one expert block's chunk
  constexpr int PF = EB == 1 ? 4 : 2;            // chunks in flight per wavefront (register-staged)
  constexpr int NTOK = FT_TOK * TT;              // tokens per workgroup
  static_assert(NTOK <= 32 && NTOK * 8 <= NWV * 64, "one flag bit and eight finalising lanes per token");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int s_flag[NTOK];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  unsigned char* wl = smem + wave * W_WAVE_BYTES;
  const int t0 = blockIdx.x * NTOK;
  const int tl = lane & 15, kq = lane >> 4;  // MFMA operand coordinates of this lane

  // activation rows of this lane, one per token tile (clamped: tail tokens recompute the last row, never stored)
  const uint16_t* xrow[TT];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) xrow[tt] = x + (size_t)min(t0 + tt * FT_TOK + tl, T - 1) * d + kq * 16;

  double zacc[TT][EB][4];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt)
#pragma unroll
    for (int b = 0; b < EB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) zacc[tt][b][r] = 0.0;

  // router-weight micro-tiles of this lane: 4 consecutive k x 4 consecutive experts each
  // (micro-tile m of a lane belongs to expert block m: expert group m*4 + lane%4, K group lane/4)
  constexpr int MT_PER_LANE = (FT_KC / 4) * (EP / 4) / 64;  // = EB
  const int n_chunks = d / FT_KC;

  // PF register stages.  Every stage load is unconditional (a chunk index past the end re-reads the last
  // chunk and is never used), so the number of loads in flight is fixed and the wait before a stage's
  // first use can leave the younger stages outstanding.
  u32x4 xa[PF][TT][2];
  float wv[PF][MT_PER_LANE][4][4];
#define GATE_LOAD_STAGE(s_, c_)                                                                         \
  {                                                                                                     \
    const int k0_ = min((c_), n_chunks - 1) * FT_KC;                                                    \
    _Pragma("unroll") for (int tt_ = 0; tt_ < TT; ++tt_) {                                              \
      xa[s_][tt_][0] = *reinterpret_cast<const u32x4*>(xrow[tt_] + k0_);                                \
      xa[s_][tt_][1] = *reinterpret_cast<const u32x4*>(xrow[tt_] + k0_ + 8);                            \
    }                                                                                                   \
    _Pragma("unroll") for (int m = 0; m < MT_PER_LANE; ++m) {                                           \
      const int eg = m * 4 + (lane & 3), kg = lane >> 2;                                                \
      _Pragma("unroll") for (int i = 0; i < 4; ++i) {                                                   \
        const float* wp = wr + (size_t)(k0_ + kg * 4 + i) * E;                                          \
        if (VEC) {                                                                                      \
          const f32x4 v = *reinterpret_cast<const f32x4*>(wp + min(eg * 4, E - 4));                     \
          const bool ok = eg * 4 < E;                                                                   \
          wv[s_][m][i][0] = ok ? v[0] : 0.f; wv[s_][m][i][1] = ok ? v[1] : 0.f;                         \
          wv[s_][m][i][2] = ok ? v[2] : 0.f; wv[s_][m][i][3] = ok ? v[3] : 0.f;                         \
        } else {                                                                                        \
          _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                               \
            const int e = eg * 4 + j;                                                                   \
            const float v = wp[min(e, E - 1)];                                                          \
            wv[s_][m][i][j] = e < E ? v : 0.f;                                                          \
          }                                                                                             \
        }                                                                                               \
      }                                                                                                 \
    }                                                                                                   \
  }

  // chunks wave, wave+NWV, ...  The LDS staging area is private to the wavefront and LDS operations of one
  // wavefront execute in order, so no barrier is needed inside this loop.
#pragma unroll
  for (int s = 0; s < PF; ++s) GATE_LOAD_STAGE(s, wave + NWV * s)
  for (int base = wave; base < n_chunks; base += NWV * PF) {
#pragma unroll
    for (int s = 0; s < PF; ++s) {
      const int c = base + NWV * s;
      const bool live = c < n_chunks;  // uniform
      bf16x8 xb[TT][2];
      f32x4 acc[TT][EB];
      if (live) {
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
          xb[tt][0] = __builtin_bit_cast(bf16x8, xa[s][tt][0]);
          xb[tt][1] = __builtin_bit_cast(bf16x8, xa[s][tt][1]);
        }
        // one expert block at a time: split its router weights into three bf16 pieces, stage them
        // K-contiguous per expert, multiply
#pragma unroll
        for (int m = 0; m < MT_PER_LANE; ++m) {
          const int egl = lane & 3, kg = lane >> 2;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            uint32_t hi[4], mid[4], lo[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float w = wv[s][m][i][j];
              hi[i] = bf16_bits_rne(w);
              const float r1 = w - __uint_as_float(hi[i] << 16);
              mid[i] = bf16_bits_rne(r1);
              const float r2 = r1 - __uint_as_float(mid[i] << 16);
              lo[i] = bf16_bits_rne(r2);
            }
            unsigned char* row = wl + (egl * 4 + j) * FT_ROW + kg * 8;
            u32x2 v;
            v.x = hi[0] | (hi[1] << 16); v.y = hi[2] | (hi[3] << 16);
            *reinterpret_cast<u32x2*>(row) = v;
            v.x = mid[0] | (mid[1] << 16); v.y = mid[2] | (mid[3] << 16);
            *reinterpret_cast<u32x2*>(row + 16 * FT_ROW) = v;
            v.x = lo[0] | (lo[1] << 16); v.y = lo[2] | (lo[3] << 16);
            *reinterpret_cast<u32x2*>(row + 2 * 16 * FT_ROW) = v;
          }
          asm volatile("" ::: "memory");  // keep the LDS reads below the LDS writes above (same wavefront: in order)
#pragma unroll
          for (int tt = 0; tt < TT; ++tt) acc[tt][m] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int p = 0; p < 3; ++p) {
              const bf16x8 wf = *reinterpret_cast<const bf16x8*>(wl + (p * 16 + tl) * FT_ROW + kq * 32 + s2 * 16);
#pragma unroll
              for (int tt = 0; tt < TT; ++tt)
                acc[tt][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, xb[tt][s2], acc[tt][m], 0, 0, 0);
            }
          asm volatile("" ::: "memory");  // ... and the next block's writes below these reads
        }
      }
      GATE_LOAD_STAGE(s, c + NWV * PF)  // refill this register stage
      if (live) {
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
          for (int b = 0; b < EB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) zacc[tt][b][r] += (double)acc[tt][b][r];
      }
    }
  }
#undef GATE_LOAD_STAGE
  lds_barrier();     // every wavefront is done with its staging area

  // ---- cross-wavefront sum of the partial logits (float64) and per-token finalisation ------------
  double* part = reinterpret_cast<double*>(smem);  // [NWV][EP][NTOK]
#pragma unroll
  for (int tt = 0; tt < TT; ++tt)
#pragma unroll
    for (int b = 0; b < EB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        part[((size_t)wave * EP + b * 16 + kq * 4 + r) * NTOK + tt * FT_TOK + tl] = zacc[tt][b][r];
  lds_barrier();
  if (tid < NTOK * 8) {
    const int tok = tid >> 3, sub = tid & 7;
    const int t = t0 + tok;
    double z[NPL];
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
      const int e = sub + 8 * i;
      double v = -INFINITY;
      if (e < E) {
        v = part[(size_t)e * NTOK + tok];
#pragma unroll
        for (int w = 1; w < NWV; ++w) v += part[((size_t)w * EP + e) * NTOK + tok];
        if (br) v += (double)br[e];
      }
      z[i] = v;
    }
    const int tc = min(t, T - 1);  // tail tokens run the same code on the last row, without storing
    float zmax = 0.f;
#pragma unroll
    for (int i = 0; i < NPL; ++i)
      if (sub + 8 * i < E) zmax = fmaxf(zmax, fabsf((float)z[i]));
    group8_steps([&](auto st) { zmax = fmaxf(zmax, group8_partner<decltype(st)::value>(zmax)); });
    bool flag = false;
    if (t < T)
      flag = finalize_group<NPL>(z, sub, E, k, renorm, GATE_MARGIN_REL * zmax, topk_idx + (size_t)tc * k, topk_w + (size_t)tc * k,
                                 probs ? probs + (size_t)tc * E : nullptr);
    if (sub == 0) s_flag[tok] = flag ? 1 : 0;
  }
  lds_barrier();

  // ---- exact recompute of the rare tokens whose ranking is within the margin -------------------
  // Each wavefront takes a contiguous K range; a load instruction covers whole router rows (lane = expert
  // quad + row slot), so that it is coalesced and many of them can be in flight: a token flagged in one
  // workgroup delays the whole kernel by the time this takes.  The products are exact in float64 and so is
  // their sum up to rounding at 2^-53, far below any gap that can decide a ranking.  The flags are turned
  // into one wave-uniform mask first (no LDS read per token).
  uint32_t flagged = (uint32_t)__ballot(lane < NTOK && s_flag[lane & (NTOK - 1)] != 0);
  flagged = __builtin_amdgcn_readfirstlane(flagged);
  constexpr int QN = EP / 4;    // expert quads per router row
  constexpr int RPI = 64 / QN;  // router rows per load instruction of a wavefront
  double* zpart = part;         // [NWV][EP]
  double* zex = part + NWV * EP;  // [EP]
  const int q = lane % QN, rs = lane / QN;
  const int rows_per_wave = d / NWV;  // d is a multiple of 64: a whole number of load instructions
  const bool qlive = q * 4 < E;
  while (flagged) {
    const int tt = __builtin_ctz(flagged);
    flagged &= flagged - 1;
    const int t = t0 + tt;
    const uint16_t* xt = x + (size_t)t * d;
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    const int r_end = (wave + 1) * rows_per_wave;
#pragma unroll 8
    for (int r = wave * rows_per_wave + rs; r < r_end; r += RPI) {
      const double xv = (double)bf16_to_f32(xt[r]);
      const float* wp = wr + (size_t)r * E + q * 4;
      float w[4] = {0.f, 0.f, 0.f, 0.f};
      if (VEC) {
        if (qlive) {  // E is a multiple of 4: q*4 + 3 < E
          const f32x4 v = *reinterpret_cast<const f32x4*>(wp);
          w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3];
        }
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (q * 4 + j < E) w[j] = wp[j];
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) a[j] = fma(xv, (double)w[j], a[j]);
    }
#pragma unroll
    for (int m = QN; m < 64; m <<= 1)
#pragma unroll
      for (int j = 0; j < 4; ++j) a[j] += shfl_xor_f64(a[j], m);
    if (rs == 0) {
#pragma unroll
      for (int j = 0; j < 4; ++j) zpart[wave * EP + q * 4 + j] = a[j];
    }
    lds_barrier();
    if (tid < E) {
      double v = zpart[tid];
#pragma unroll
      for (int w = 1; w < NWV; ++w) v += zpart[w * EP + tid];
      zex[tid] = v + (br ? (double)br[tid] : 0.0);
    }
    lds_barrier();
    if (tid < 8) {
      double z[NPL];
#pragma unroll
      for (int i = 0; i < NPL; ++i) z[i] = (tid + 8 * i) < E ? zex[tid + 8 * i] : -INFINITY;
      finalize_group<NPL>(z, tid, E, k, renorm, 0.f, topk_idx + (size_t)t * k, topk_w + (size_t)t * k,
                          probs ? probs + (size_t)t * E : nullptr);
    }
    lds_barrier();
  }
}

template <int EB>
int32_t launch_fast(const moe_config* cfg, const void* x, const float* w_router, const float* b_router,
                    int32_t* topk_idx, float* topk_w, float* probs, hipStream_t s) {
  constexpr int EP = EB * 16;
  constexpr int NWV = gate_waves<EB>();
  const size_t w_bytes = (size_t)NWV * 3 * 16 * FT_ROW;
  // two token tiles per workgroup for narrow routers once that still leaves a workgroup for every CU
  constexpr int TT_MAX = EB == 1 ? 2 : 1;
  const int tt = (TT_MAX == 2 && cfg->T >= 2 * FT_TOK * 256) ? 2 : 1;  // (256 CUs)
  const size_t z_bytes = (size_t)NWV * EP * FT_TOK * tt * sizeof(double) + 256;
  const size_t shmem = w_bytes > z_bytes ? w_bytes : z_bytes;
  const bool vec = cfg->E % 4 == 0 && ((uintptr_t)w_router & 15) == 0;
  auto kern = tt == 2 ? (vec ? gate_mfma_kernel<EB, true, TT_MAX> : gate_mfma_kernel<EB, false, TT_MAX>)
                      : (vec ? gate_mfma_kernel<EB, true, 1> : gate_mfma_kernel<EB, false, 1>);
  if (shmem > 65536) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
    if (e != hipSuccess) return check_hip(e, "hipFuncSetAttribute(gate LDS)");
  }
  hipLaunchKernelGGL(kern, dim3((cfg->T + FT_TOK * tt - 1) / (FT_TOK * tt)), dim3(NWV * 64), shmem, s, (const uint16_t*)x, w_router,
                     b_router, cfg->T, cfg->d_model, cfg->E, cfg->k, cfg->renormalize, topk_idx, topk_w, probs);
  return check_hip(hipGetLastError(), "gate launch");
}


// ------------------------------------------------------------------------------------------------
// Fast path on a pre-split router (moe_pack_router): the HBM-rate gate.
//
// The split of the float32 router into three bfloat16 pieces does not depend on the tokens, so it is done once,
// outside the hot path, into the order the MFMA reads its operand in: rows of the packed matrix are
// (piece, expert) pairs, row = piece * E + expert, padded with zero rows to FR blocks of 32; the contraction
// index runs in stages of KC = 16 G values, and inside a stage the lower 32 lanes of a wavefront hold its
// first KC/2 values and the upper 32 lanes the others (a dot product does not care about the order, as long as
// both operands use the same one): that way a lane's share of a token row is one contiguous run of KC bytes and
// a wavefront's loads of one stage cover whole cache lines of every token row.  A fragment (stage, sub-step,
// row block) is 1 KB, contiguous, in that order.
//
// One workgroup = NT = 32 NB tokens, eight wavefronts that split the contraction index in runs of a few stages.  A wavefront multiplies v_mfma_f32_32x32x16_bf16 tiles, router rows x tokens, and
// every product is exact in float32 (a bfloat16 piece times a bfloat16 activation), so the only rounding is the
// float32 accumulation over the wavefront's share of the contraction index; the eight partial sums and the three
// pieces of an expert meet in float64 through LDS.  No staging through LDS on the way in, no conversion in the
// loop: the loop is loads and MFMAs, and the kernel runs at the rate the token rows arrive from HBM.
//
// Ranking must equal the ranking of the exactly computed logits.  The partial sums carry errors of about
// 2^-24 times their own magnitude, so a token is marked when two neighbours among its k+1 leading logits are
// closer than 2^-15 times the largest sum over the wavefronts of |partial logit| of that token (a margin that
// scales with the data; about 1e-4 for inputs of unit variance): the mark is the sign bit of its first gate
// weight, and gate_fix_kernel, launched behind this kernel, recomputes the marked tokens with float64
// accumulation of the exact products, from the float32 router itself.
#ifndef GATE_REL_MARGIN_VALUE
#define GATE_REL_MARGIN_VALUE (1.0f / 32768.0f)
#endif
constexpr float GATE_REL_MARGIN = GATE_REL_MARGIN_VALUE;
constexpr int GP_WAVES = 8;

__host__ __device__ constexpr int gate_frags(int E) { return (3 * E + 31) / 32; }        // row blocks of the packed router
__host__ __device__ constexpr int gate_substeps(int FR) { return FR <= 3 ? 4 : 2; }      // MFMA sub-steps per stage

// one thread per 16-byte piece of the packed router
__global__ __launch_bounds__(256) void pack_router_kernel(const float* __restrict__ wr, uint16_t* __restrict__ dst, int d, int E,
                                                          int FR, int G) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t total = (size_t)(d / (16 * G)) * G * FR * 64;
  if (i >= total) return;
  const int lane = (int)(i % 64);
  const size_t frag = i / 64;
  const int fr = (int)(frag % FR), s = (int)((frag / FR) % G);
  const size_t c = frag / ((size_t)FR * G);
  const int row = 32 * fr + (lane & 31), h = lane >> 5;
  const int piece = row / E, e = row - piece * E;
  const size_t k0 = c * (16 * G) + (size_t)(8 * G) * h + 8 * s;
  uint32_t out[4] = {0u, 0u, 0u, 0u};
  if (piece < 3) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float w = wr[(k0 + j) * E + e];
      const uint32_t hi = bf16_bits_rne(w);
      const float r1 = w - __uint_as_float(hi << 16);      // exact: the leading 8 bits of the significand are gone
      const uint32_t mid = bf16_bits_rne(r1);
      const float r2 = r1 - __uint_as_float(mid << 16);    // exact; at most 8 significant bits are left
      const uint32_t lo = bf16_bits_rne(r2);
      const uint32_t v = piece == 0 ? hi : piece == 1 ? mid : lo;
      out[j >> 1] |= v << (16 * (j & 1));
    }
  }
  *reinterpret_cast<u32x4*>(dst + i * 8) = u32x4{out[0], out[1], out[2], out[3]};
}

typedef float f32x16 __attribute__((ext_vector_type(16)));

// f(integral_constant<int, 0>{}), ..., f(integral_constant<int, N - 1>{}), unrolled
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// One token's logits with float64 accumulation of the exact products of the float32 router and the activations,
// then softmax and ranking on those values: the whole workgroup of GP_WAVES wavefronts works on the token.  Every
// wavefront takes a contiguous range of router rows; a load instruction covers whole rows (lane = expert quad + row
// slot) and sixteen of them are in flight.  lds: (GP_WAVES + 1) * 64 doubles; the caller synchronises before.
__device__ __forceinline__ void exact_token(const uint16_t* __restrict__ x, const float* __restrict__ wr, const float* __restrict__ br,
                                            int t, int d, int E, int k, int renorm, int32_t* __restrict__ topk_idx,
                                            float* __restrict__ topk_w, float* __restrict__ probs, double* lds) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // expert quads per router row (a power of two that covers E) and router rows per wave-wide load instruction
  const int QN = E <= 4 ? 1 : E <= 8 ? 2 : E <= 16 ? 4 : E <= 32 ? 8 : 16, RPI = 64 / QN;
  double* zpart = lds;                  // [GP_WAVES][64]
  double* zex = lds + GP_WAVES * 64;    // [64]
  const int q = lane % QN, rs = lane / QN;
  const int rows_per_wave = d / GP_WAVES;   // d is a multiple of 64
  const bool vec = (E & 3) == 0 && (reinterpret_cast<uintptr_t>(wr) & 15) == 0;
  const uint16_t* xt = x + (size_t)t * d;
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  // All loads of a batch are issued before the first is used, and the trip count is the same for every lane (rows
  // past the wavefront's range re-read its first row and are multiplied by zero): a loop that can leave early
  // makes the compiler wait for every load where it stands, and the token then costs one memory latency per
  // router row instead of one per batch.
  const int r_begin = wave * rows_per_wave, r_end = r_begin + rows_per_wave;
  const int n_it = (rows_per_wave + RPI - 1) / RPI;
  const bool q_live = q * 4 < E;
  const int last = q_live ? min(3, E - 1 - q * 4) : 0;   // scalar loads of a ragged last quad stay inside the row
  auto rows = [&](auto is_vec, auto batch) {
    constexpr int BATCH = decltype(batch)::value;
    for (int it0 = 0; it0 < n_it; it0 += BATCH) {
      float w4[BATCH][4];
      uint16_t xb[BATCH];
#pragma unroll
      for (int j = 0; j < BATCH; ++j) {
        const int r = r_begin + rs + (it0 + j) * RPI;
        const int rc = r < r_end ? r : r_begin;
        const float* wq = q_live ? wr + (size_t)rc * E + q * 4 : wr;   // quads past the last expert read the first row
        if constexpr (decltype(is_vec)::value) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(wq);
          w4[j][0] = v[0]; w4[j][1] = v[1]; w4[j][2] = v[2]; w4[j][3] = v[3];
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c) w4[j][c] = wq[min(c, last)];
        }
        xb[j] = xt[rc];
      }
#pragma unroll
      for (int j = 0; j < BATCH; ++j) {
        const int r = r_begin + rs + (it0 + j) * RPI;
        const double xd = r < r_end ? (double)bf16_to_f32(xb[j]) : 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) a[c] = fma(xd, (q * 4 + c < E) ? (double)w4[j][c] : 0.0, a[c]);
      }
    }
  };
  if (vec) rows(std::true_type{}, std::integral_constant<int, 16>{});
  else rows(std::false_type{}, std::integral_constant<int, 16>{});
  for (int m = QN; m < 64; m <<= 1)
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] += shfl_xor_f64(a[j], m);
  if (rs == 0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) zpart[wave * 64 + q * 4 + j] = a[j];
  }
  __syncthreads();
  if (tid < E) {
    double v = zpart[tid];
#pragma unroll
    for (int w = 1; w < GP_WAVES; ++w) v += zpart[w * 64 + tid];
    zex[tid] = v + (br ? (double)br[tid] : 0.0);
  }
  __syncthreads();
  if (tid < 8) {
    double z[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] = (tid + 8 * i) < E ? zex[tid + 8 * i] : -INFINITY;
    finalize_group<8>(z, tid, E, k, renorm, 0.f, topk_idx + (size_t)t * k, topk_w + (size_t)t * k,
                      probs ? probs + (size_t)t * E : nullptr);
  }
}

// Recomputes the tokens that gate_packed_kernel marked (sign bit of the first gate weight): one workgroup looks at
// FIX_TOKENS tokens and works through the marked ones (almost always none, rarely one), replacing indices, weights
// and probabilities.  Launched behind every gate_packed_kernel: inside that kernel a marked token would hold up its
// whole workgroup, and with it the kernel, for the time of a chain of dependent loads.
constexpr int FIX_TOKENS = 64;
__global__ __launch_bounds__(GP_WAVES * 64) void gate_fix_kernel(const uint16_t* __restrict__ x, const float* __restrict__ wr,
                                                                 const float* __restrict__ br, int T, int d, int E, int k, int renorm,
                                                                 int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                                                 float* __restrict__ probs) {
  __shared__ double lds[(GP_WAVES + 1) * 64];
  const int lane = threadIdx.x & 63;
  const int t0 = blockIdx.x * FIX_TOKENS;
  static_assert(FIX_TOKENS == 64, "one ballot");
  const int t = t0 + lane;
  unsigned long long todo = __ballot(t < T && (__float_as_uint(topk_w[(size_t)min(t, T - 1) * k]) >> 31) != 0);
  while (todo) {
    const int st = __builtin_ctzll(todo);
    todo &= todo - 1;
    __syncthreads();
    exact_token(x, wr, br, t0 + st, d, E, k, renorm, topk_idx, topk_w, probs, lds);
  }
}

// What follows the contraction in the gate kernels on a packed router: acc[nb][fr] holds this wavefront's partial
// sums (router rows x tokens, the MFMA's accumulator layout) for the NT = 32 NB tokens from t0 on.  The partial sums
// of the eight wavefronts and the three pieces of every expert meet in float64 through LDS (smem: room for the
// partial-sum matrices), then softmax, ranking and the margin test per token; tokens within the margin are
// marked for gate_fix_kernel.
template <int FR, int NB>
__device__ __forceinline__ void gate_finish(f32x16 (&acc)[NB][FR], unsigned char* smem, int t0, const float* __restrict__ br, int T,
                                            int E, int k, int renorm, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                            float* __restrict__ probs) {
  constexpr int NT = 32 * NB, RW = 32 * FR;
  constexpr int STRIDE = NT + 8;  // floats between the rows of a partial-sum matrix (conflict-free reads and writes)
  constexpr int NPL = (32 * FR / 3 + 7) / 8;  // logits per lane of an 8-lane group (covers every E of this FR)
  // all eight partial-sum matrices in LDS at once, or four and two rounds
  constexpr bool TWO_ROUNDS = (size_t)GP_WAVES * RW * STRIDE * 4 > 150 * 1024;
  constexpr int SLOTS = TWO_ROUNDS ? GP_WAVES / 2 : GP_WAVES;
  float* part = reinterpret_cast<float*>(smem);  // [SLOTS][RW][STRIDE]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tok = lane & 31, h = lane >> 5;
  // ---- the partial sums meet in LDS: part[slot][row][token] -------------------------------------
  auto put = [&](int slot) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int fr = 0; fr < FR; ++fr)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = 32 * fr + 8 * (v >> 2) + 4 * h + (v & 3);
          part[((size_t)slot * RW + row) * STRIDE + 32 * nb + tok] = acc[nb][fr][v];
        }
  };
  if constexpr (TWO_ROUNDS) {
    // the upper four wavefronts hand their sums to the lower four (one float32 addition: 2^-24 of a partial sum)
    if (wave >= SLOTS) put(wave - SLOTS);
    __syncthreads();
    if (wave < SLOTS) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int fr = 0; fr < FR; ++fr)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int row = 32 * fr + 8 * (v >> 2) + 4 * h + (v & 3);
            acc[nb][fr][v] += part[((size_t)wave * RW + row) * STRIDE + 32 * nb + tok];
          }
    }
    __syncthreads();
    if (wave < SLOTS) put(wave);
  } else {
    put(wave);
  }
  __syncthreads();

  // ---- per token: float64 sum over wavefronts and pieces, float32 softmax, ranking, margin test ----------
  for (int base = 0; base < NT; base += GP_WAVES * 8) {
    const int slot_tok = base + (tid >> 3), sub = tid & 7;
    const int t = t0 + slot_tok;
    if (slot_tok < NT) {   // (uniform per 8-lane group)
      double z[NPL];
      float zabs = 0.f;
#pragma unroll
      for (int i = 0; i < NPL; ++i) {
        const int e = sub + 8 * i;
        double v = -INFINITY;
        if (e < E) {
          v = 0.0;
          float a = 0.f;
          for (int w = 0; w < SLOTS; ++w) {
            const float* pw = part + ((size_t)w * RW + e) * STRIDE + slot_tok;
            const double pz = (double)pw[0] + (double)pw[(size_t)E * STRIDE] + (double)pw[(size_t)2 * E * STRIDE];
            v += pz;
            a += fabsf((float)pz);
          }
          zabs = fmaxf(zabs, a);
          if (br) v += (double)br[e];
        }
        z[i] = v;
      }
      group8_steps([&](auto st) { zabs = fmaxf(zabs, group8_partner<decltype(st)::value>(zabs)); });
      const int tc = min(t, T - 1);
      if (t < T)
        finalize_group<NPL>(z, sub, E, k, renorm, GATE_REL_MARGIN * zabs, topk_idx + (size_t)tc * k, topk_w + (size_t)tc * k,
                            probs ? probs + (size_t)tc * E : nullptr, true);
    }
  }

}

template <int FR, int NB>
__global__ __launch_bounds__(GP_WAVES * 64) void gate_packed_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ wp,
                                                                    const float* __restrict__ wr, const float* __restrict__ br, int T,
                                                                    int d, int E, int k, int renorm, int32_t* __restrict__ topk_idx,
                                                                    float* __restrict__ topk_w, float* __restrict__ probs) {
  constexpr int G = gate_substeps(FR), KC = 16 * G, NT = 32 * NB;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tok = lane & 31, h = lane >> 5;
  const int t0 = blockIdx.x * NT;
  const int n_stages = d / KC;

  // this lane's run of every token row (tail tokens recompute the last row and are never stored)
  const uint16_t* xrow[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) xrow[nb] = x + (size_t)min(t0 + 32 * nb + tok, T - 1) * d + (KC / 2) * h;
  const uint16_t* wlane = wp + lane * 8;

  f32x16 acc[NB][FR];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int fr = 0; fr < FR; ++fr)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[nb][fr][v] = 0.f;

  // PF register stages in flight.  Every stage load is unconditional (a stage index past the end re-reads the
  // last stage) and every stage is multiplied, with the token fragments of a stage past the end replaced by
  // zeros (which add nothing): loads and uses then sit in straight-line code, the compiler can neither sink a
  // load into a branch next to its use nor merge the stages' registers, and a scheduling barrier after each
  // group of loads keeps them ahead of the multiplications of the older stages.
  constexpr int STAGE_REGS = (NB + FR) * G * 4;
  constexpr int PF = STAGE_REGS <= 32 ? 4 : STAGE_REGS <= 48 ? 3 : 2;
  u32x4 xs[PF][NB][G], ws[PF][G][FR];
  auto load_stage = [&](auto b_tag, int c) {
    constexpr int b = decltype(b_tag)::value;
    const int cc = min(c, n_stages - 1);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int s = 0; s < G; ++s) xs[b][nb][s] = *reinterpret_cast<const u32x4*>(xrow[nb] + (size_t)cc * KC + 8 * s);
#pragma unroll
    for (int s = 0; s < G; ++s)
#pragma unroll
      for (int fr = 0; fr < FR; ++fr)
        ws[b][s][fr] = *reinterpret_cast<const u32x4*>(wlane + (((size_t)cc * G + s) * FR + fr) * 512);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&](auto b_tag, int c) {
    constexpr int b = decltype(b_tag)::value;
    const uint32_t keep = c < n_stages ? 0xffffffffu : 0u;   // (uniform)
#pragma unroll
    for (int s = 0; s < G; ++s)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const u32x4 xv = xs[b][nb][s] & keep;
#pragma unroll
        for (int fr = 0; fr < FR; ++fr)
          acc[nb][fr] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ws[b][s][fr]),
                                                                __builtin_bit_cast(bf16x8, xv), acc[nb][fr], 0, 0, 0);
      }
    __builtin_amdgcn_sched_barrier(0);
  };
  // wavefront w takes stages w PF .. w PF + PF - 1, then those 8 PF further on, ...: the PF stages it has in flight
  // are one contiguous run of every token row (PF KC values), which is what DRAM pages and cache lines like
  static_for<PF>([&](auto j) { load_stage(j, wave * PF + decltype(j)::value); });
  for (int c = wave * PF; c < n_stages; c += PF * GP_WAVES)
    static_for<PF>([&](auto j) {
      constexpr int jj = decltype(j)::value;
      multiply(j, c + jj);
      load_stage(j, c + jj + PF * GP_WAVES);
    });

  gate_finish<FR, NB>(acc, smem, t0, br, T, E, k, renorm, topk_idx, topk_w, probs);
}

template <int FR, int NB>
int32_t launch_packed(const moe_config* cfg, const void* x, const void* packed, const float* w_router, const float* b_router,
                      int32_t* topk_idx, float* topk_w, float* probs, hipStream_t s) {
  constexpr int NT = 32 * NB, RW = 32 * FR, STRIDE = NT + 8;
  constexpr bool TWO_ROUNDS = (size_t)GP_WAVES * RW * STRIDE * 4 > 150 * 1024;
  constexpr size_t shmem = (size_t)(TWO_ROUNDS ? GP_WAVES / 2 : GP_WAVES) * RW * STRIDE * 4;
  static_assert(shmem <= 160 * 1024, "partial sums do not fit the LDS");
  auto kern = gate_packed_kernel<FR, NB>;
  if (shmem > 65536) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
    if (e != hipSuccess) return check_hip(e, "hipFuncSetAttribute(gate LDS)");
  }
  hipLaunchKernelGGL(kern, dim3((cfg->T + NT - 1) / NT), dim3(GP_WAVES * 64), shmem, s, (const uint16_t*)x, (const uint16_t*)packed,
                     w_router, b_router, cfg->T, cfg->d_model, cfg->E, cfg->k, cfg->renormalize, topk_idx, topk_w, probs);
  hipLaunchKernelGGL(gate_fix_kernel, dim3((cfg->T + FIX_TOKENS - 1) / FIX_TOKENS), dim3(GP_WAVES * 64), 0, s, (const uint16_t*)x,
                     w_router, b_router, cfg->T, cfg->d_model, cfg->E, cfg->k, cfg->renormalize, topk_idx, topk_w, probs);
  return check_hip(hipGetLastError(), "gate launch");
}

}  // namespace

// A step of one token: gate and dispatch tables from one kernel (bf16 activations: the layer then needs no
// dispatched copy of the token).
bool gate_dispatch_one_token_applies(const moe_config* cfg, const float* w_router) {
  return cfg->T == 1 && cfg->dtype == MOE_BF16 && gate_few_applies(cfg, w_router);
}
// Gate and dispatch tables of a step of few tokens through slices of the contraction index; scratch: room for the partial logits.
static bool gate_slices_fit(const moe_config* cfg, const float* w_router, size_t scratch_bytes) {
  const GateSlices p = plan_gate_slices(cfg, w_router, scratch_bytes);
  return p.slices >= 1 && p.logits <= GR_LOGITS;
}
bool gate_dispatch_slices_applies(const moe_config* cfg, const float* w_router, size_t scratch_bytes) {
  if (!tuning(MOE_TUNE_FEW_TOKEN_KERNELS) || cfg->dtype != MOE_BF16 || cfg->T < 1 || cfg->T > GR_MAX_T ||
      (int64_t)cfg->T * cfg->k > GR_THREADS)
    return false;
  // (measured: see gate_rank_kernel; one token on a small router: one workgroup does it all)
  if (cfg->T > 96 && cfg->d_model < 1536) return false;
  if (gate_dispatch_one_token_applies(cfg, w_router) && (int64_t)cfg->d_model * cfg->E < 131072) return false;
  return gate_slices_fit(cfg, w_router, scratch_bytes);
}
int32_t launch_gate_dispatch_slices(const moe_config* cfg, const void* x, const float* w_router, const float* b_router, int32_t* topk_idx,
                                    float* topk_w, int32_t* counts, int32_t* offsets, int32_t* a2r, int32_t* r2a, int32_t* clear8,
                                    void* scratch, size_t scratch_bytes, hipStream_t s) {
  const GateSlices p = plan_gate_slices(cfg, w_router, scratch_bytes);
  const int32_t st = launch_gate_parts(cfg, p, x, w_router, (double*)scratch, s);
  if (st != MOE_OK) return st;
  const int E = cfg->E;
  auto kern = gate_few_applies(cfg, w_router)
                  ? (E <= 16 ? gate_rank_kernel<2, true> : E <= 32 ? gate_rank_kernel<4, true> : gate_rank_kernel<8, true>)
                  : E <= 16 ? gate_rank_kernel<2, false> : E <= 32 ? gate_rank_kernel<4, false> : E <= 64 ? gate_rank_kernel<8, false>
                  : E <= 128 ? gate_rank_kernel<16, false> : gate_rank_kernel<32, false>;
  size_t shmem = ((size_t)p.logits + 8 * (size_t)cfg->T) * sizeof(double);
  if (shmem < sizeof(OneTables)) shmem = sizeof(OneTables);
  if (shmem > 48 * 1024) {
    const hipError_t err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
    if (err != hipSuccess) return check_hip(err, "hipFuncSetAttribute(gate LDS)");
  }
  hipLaunchKernelGGL(kern, dim3(1), dim3(GR_THREADS), shmem, s, (const double*)scratch, b_router, cfg->T, E, cfg->k, moe_capacity(cfg),
                     cfg->renormalize, p.slices, topk_idx, topk_w, counts, offsets, a2r, r2a, clear8);
  return check_hip(hipGetLastError(), "gate launch");
}

// The slices alone, for a one-token step whose first product ranks (expert_gemv_ranked_applies): their number, 0 where the step does
// not take slices.
int gate_parts_one_token(const moe_config* cfg, const float* w_router, size_t scratch_bytes) {
  if (!tuning(MOE_TUNE_FEW_TOKEN_KERNELS) || cfg->dtype != MOE_BF16 || cfg->T != 1 || !gate_slices_fit(cfg, w_router, scratch_bytes)) return 0;
  return plan_gate_slices(cfg, w_router, scratch_bytes).slices;
}
int32_t launch_gate_parts_one_token(const moe_config* cfg, const void* x, const float* w_router, double* part, size_t scratch_bytes, hipStream_t s) {
  return launch_gate_parts(cfg, plan_gate_slices(cfg, w_router, scratch_bytes), x, w_router, part, s);
}

int32_t launch_gate_dispatch_one_token(const moe_config* cfg, const void* x, const float* w_router, const float* b_router,
                                       int32_t* topk_idx, float* topk_w, int32_t* counts, int32_t* offsets, int32_t* a2r,
                                       int32_t* r2a, int32_t* clear8, hipStream_t s) {
  return launch_few<uint16_t>(cfg, x, w_router, b_router, topk_idx, topk_w, nullptr, s, counts, offsets, a2r, r2a, clear8);
}

// bfloat16 activations, up to 64 experts: where the float64 kernel takes over from the one that splits the router into
// bfloat16 pieces.  Splitting costs every workgroup of 16 tokens the whole router on the vector ALU, and an element-wise read
// of it where E is no multiple of 4; a float64 MFMA costs 32 times a bfloat16 one, which grows with d, and its workgroups
// (16 tokens, one per CU) run in rounds of 4096 tokens.  Measured on MI355X (us, split / float64, means over four inputs):
//   16 experts, d 2048: T 4096 14.5 / 12.0, T 16384 27 / 33, and two token tiles per workgroup take over from T 8192, so up
//     to 16 experts stay with the split; below 1024 tokens too: 24 experts, d 2048, T 300 13.3 / 15.8;
//   24 experts: d 1024 T 1024 11 / 11, T 4096 13 / 12, T 16384 39 / 34; d 1536 T 4096 18 / 14; d 2048 T 1536 16 / 17, T 4097
//     26 / 29; d 4096 T 1024 25 / 27, T 4097 40 / 50: float64 up to d 1536;
//   64 experts: d 1024 T 4096 26 / 17, T 4097 32 / 30; d 2048 T 1024 27 / 24, T 4096 49 / 26, T 4097 49 / 47; d 4096 T 4096
//     70 / 43, T 4097 80 / 81, T 8193 113 / 119, T 10000 120 / 121: float64, but not for a last round that is nearly empty
//     where d is above 2048 (48 experts, d 3072, T 4097: 58 / 62);
//   E no multiple of 4: 31 experts, d 2048, T 1024 43 / 18; 63 experts, d 4096, T 4096 156 / 81: float64.
bool gate_f64_pays(const moe_config* cfg) {
  const int T = cfg->T, d = cfg->d_model, E = cfg->E;
  if (E <= 16 || T < 1024) return false;
  if (E % 4) return true;
  if (E <= 32) return d <= 1536;
  const int last = T % 4096;  // tokens of the last round
  return d <= 2048 || T <= 4096 || last == 0 || last > 1024;
}

int32_t launch_gate(const moe_config* cfg, const void* x, const float* w_router, const float* b_router,
                    int32_t* topk_idx, float* topk_w, float* probs, hipStream_t s) {
  if (cfg->T == 0) return MOE_OK;
  if (gate_few_applies(cfg, w_router)) {
    if (cfg->dtype == MOE_BF16) return launch_few<uint16_t>(cfg, x, w_router, b_router, topk_idx, topk_w, probs, s);
    return launch_few<float>(cfg, x, w_router, b_router, topk_idx, topk_w, probs, s);
  }
  if (cfg->dtype == MOE_BF16 && cfg->E <= 64 && !gate_f64_pays(cfg)) {
    if (cfg->E <= 16) return launch_fast<1>(cfg, x, w_router, b_router, topk_idx, topk_w, probs, s);
    if (cfg->E <= 32) return launch_fast<2>(cfg, x, w_router, b_router, topk_idx, topk_w, probs, s);
    return launch_fast<4>(cfg, x, w_router, b_router, topk_idx, topk_w, probs, s);
  }
  if (cfg->dtype == MOE_BF16) return launch_f64<uint16_t>(cfg, x, w_router, b_router, topk_idx, topk_w, probs, s);
  return launch_f64<float>(cfg, x, w_router, b_router, topk_idx, topk_w, probs, s);
}

// The pre-split router serves bfloat16 activations and up to 64 experts (3 E rows in at most six blocks of 32).
size_t router_pack_bytes(int d_model, int E) {
  if (E < 1 || E > 64 || d_model < 64 || d_model % 64) return 0;
  return (size_t)d_model * gate_frags(E) * 64;   // d/KC stages x G sub-steps x FR blocks x 1 KB
}

bool gate_packed_applies(const moe_config* cfg, const float* w_router) {
  return cfg->dtype == MOE_BF16 && cfg->E <= 64 && !gate_few_applies(cfg, w_router);
}
// Inside a layer the packed router is used where it measured faster than the kernels that need no preparation: long token
// streams (from about 64 M activation elements; below, narrow routers are bound by their chain of dependent steps and by
// the second launch that recomputes the near-ties), and, for more than 16 experts,
//  - beyond the float64 kernel's first round of 4096 tokens, except for the cheapest routers (us, float64 / packed with its
//    second launch, means over four inputs: 64 experts, d 2048: T 4096 26 / 35, T 4097 47 / 35, T 6144 47 / 36, T 8191 47 / 43,
//    T 32768 177 / 102; d 1024: T 4097 30 / 29, T 8191 29 / 28; 24 experts, d 2048: T 4097 29 / 23, T 16384 56 / 40; d 512:
//    T 4097 12 / 16, T 8192 13 / 16, T 16384 21 / 22, T 32768 38 / 37);
//  - from 1024 tokens where the router is wide and its rows cannot be read four at a time (63 experts, d 2048, T 2048 46 / 38,
//    d 4096, T 1536 80 / 46) or the float64 sums are long and the tokens few (48 experts, d 3072, T 1024 32 / 24; 40 experts,
//    d 4096, T 3072 42 / 37; but 64 experts, d 4096, T 4096 43 / 50).
bool gate_packed_pays(const moe_config* cfg) {
  const int T = cfg->T, d = cfg->d_model, E = cfg->E;
  if ((int64_t)T * d >= ((int64_t)1 << 26)) return true;
  if (E <= 16) return false;
  if (T > 4096) return d >= 1024 || E > 32 || T >= 16384;
  return T >= 1024 && E > 32 && ((E % 4 != 0 && d >= 1024) || (d >= 3072 && (T < 2048 || E <= 40)));
}

int32_t launch_gate_packed(const moe_config* cfg, const void* x, const void* packed, const float* w_router, const float* b_router,
                           int32_t* topk_idx, float* topk_w, float* probs, hipStream_t s) {
  if (cfg->T == 0) return MOE_OK;
  const int FR = gate_frags(cfg->E);
  // tokens per workgroup: as many 32-token blocks as still give every compute unit a workgroup (each workgroup
  // reads the whole packed router once, from L2)
  const int forced = tuning(MOE_TUNE_GATE_TOKENS);
  auto wgs = [&](int nb) { return forced ? (forced == 32 * nb ? 1 << 20 : 0) : (cfg->T + 32 * nb - 1) / (32 * nb); };
#define MOE_GATE_PACKED(fr, nb) return launch_packed<fr, nb>(cfg, x, packed, w_router, b_router, topk_idx, topk_w, probs, s)
  switch (FR) {
    case 1:
      if (wgs(4) >= 256) MOE_GATE_PACKED(1, 4);
      if (wgs(2) >= 256) MOE_GATE_PACKED(1, 2);
      MOE_GATE_PACKED(1, 1);
    case 2:
      if (wgs(2) >= 256) MOE_GATE_PACKED(2, 2);
      MOE_GATE_PACKED(2, 1);
    case 3: MOE_GATE_PACKED(3, 1);
    case 4: MOE_GATE_PACKED(4, 1);
    case 5: MOE_GATE_PACKED(5, 1);
    case 6: MOE_GATE_PACKED(6, 1);
  }
#undef MOE_GATE_PACKED
  return fail(MOE_ERR_UNSUPPORTED, "packed router: E=%d has no kernel", cfg->E);
}

// The gate of a layer: on the pre-split router when the weights carry one and it applies.
int32_t launch_gate_of(const moe_config* cfg, const moe_weights* w, const void* x, int32_t* topk_idx, float* topk_w, float* probs,
                       hipStream_t s) {
  if (w->w_router_packed && gate_packed_applies(cfg, w->w_router) && gate_packed_pays(cfg))
    return launch_gate_packed(cfg, x, w->w_router_packed, w->w_router, w->b_router, topk_idx, topk_w, probs, s);
  return launch_gate(cfg, x, w->w_router, w->b_router, topk_idx, topk_w, probs, s);
}

}  // namespace moesys

using namespace moesys;

extern "C" int32_t moe_gate(const moe_config* cfg, const void* x, const float* w_router,
                            const float* b_router, int32_t* topk_idx, float* topk_w, float* probs,
                            void* stream) {
  int32_t st = moe_config_check(cfg);
  if (st != MOE_OK) return st;
  if (cfg->T > 0 && (!x || !w_router || !topk_idx || !topk_w))
    return fail(MOE_ERR_INVALID_ARG, "moe_gate: x, w_router, topk_idx and topk_w must be non-NULL");
  return launch_gate(cfg, x, w_router, b_router, topk_idx, topk_w, probs, (hipStream_t)stream);
}

// Which kernel moe_gate takes (packed: moe_gate_packed where it pays) for 16-byte aligned weights, and a layer that neither cuts the
// contraction index into slices nor has one token (moe_test_layer_routing): for the tests of the rules above.  Host only; not part
// of the interface in moesys.h.
extern "C" const char* moe_test_gate_kernel(const moe_config* cfg, int32_t packed) {
  if (moe_config_check(cfg) != MOE_OK) return "";
  if (packed && gate_packed_applies(cfg, nullptr) && gate_packed_pays(cfg)) return "packed";
  if (gate_few_applies(cfg, nullptr)) return "few";
  return cfg->dtype == MOE_BF16 && cfg->E <= 64 && !gate_f64_pays(cfg) ? "split" : "float64";
}

extern "C" size_t moe_router_pack_bytes(int32_t d_model, int32_t E) { return router_pack_bytes(d_model, E); }

extern "C" int32_t moe_pack_router(const float* w_router, void* packed, int32_t d_model, int32_t E, void* stream) {
  const size_t bytes = router_pack_bytes(d_model, E);
  if (!bytes) return fail(MOE_ERR_UNSUPPORTED, "moe_pack_router: d_model=%d (multiple of 64) and E=%d (1..64) only", d_model, E);
  if (!w_router || !packed || ((uintptr_t)packed & 15)) return fail(MOE_ERR_INVALID_ARG, "moe_pack_router: NULL or misaligned pointer");
  const int FR = gate_frags(E), G = gate_substeps(FR);
  const size_t pieces = bytes / 16;
  hipLaunchKernelGGL(pack_router_kernel, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, (hipStream_t)stream, w_router,
                     (uint16_t*)packed, d_model, E, FR, G);
  return check_hip(hipGetLastError(), "router pack launch");
}

extern "C" int32_t moe_gate_packed(const moe_config* cfg, const void* x, const float* w_router, const float* b_router,
                                   const void* w_router_packed, int32_t* topk_idx, float* topk_w, float* probs, void* stream) {
  int32_t st = moe_config_check(cfg);
  if (st != MOE_OK) return st;
  if (cfg->T > 0 && (!x || !w_router || !w_router_packed || !topk_idx || !topk_w))
    return fail(MOE_ERR_INVALID_ARG, "moe_gate_packed: x, w_router, w_router_packed, topk_idx and topk_w must be non-NULL");
  if (cfg->dtype != MOE_BF16 || cfg->E > 64)
    return fail(MOE_ERR_UNSUPPORTED, "moe_gate_packed: bf16 activations and at most 64 experts (use moe_gate)");
  if (!gate_packed_applies(cfg, w_router))   // steps of very few tokens: one workgroup per token on the float32 router
    return launch_gate(cfg, x, w_router, b_router, topk_idx, topk_w, probs, (hipStream_t)stream);
  return launch_gate_packed(cfg, x, w_router_packed, w_router, b_router, topk_idx, topk_w, probs, (hipStream_t)stream);
}
