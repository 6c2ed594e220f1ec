// Internal helpers shared by the library's translation units (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "moesys.h"

namespace moesys {

// Records msg as this thread's last error and returns st.
int32_t fail(int32_t st, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
int32_t check_hip(hipError_t e, const char* what);

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline size_t elem_size(int32_t dtype) { return dtype == MOE_BF16 ? 2 : 4; }

// Current value of a moe_tuning_key (moe_set_tuning).
int32_t tuning(int32_t key);

// Upper bound of dispatched rows: min(k*T, E*C).
int64_t max_rows(const moe_config* cfg);

// Whether the expert weights that one call reads are more than the last-level cache (256 MB) keeps for the next call; every
// expert can be active, at most one per assignment.  Kernels in which no other workgroup reads the same weights then load
// them non-temporally: a loop of nothing but such loads into LDS reaches 7.1 TB/s, with ordinary ones 6.4, and what the
// layer's other kernels use (router, tokens, activations) stays cached.  Weights that fit are read faster through the cache.
// The line: whole layers of 2 tokens per expert on three token sets in turn, 8 to 32 experts, d_model 1024 to 4096, time with
// ordinary / with non-temporal loads: up to 270 MB 0.80 to 0.97, 285 to 302 MB 0.89 to 1.02, 315 to 380 MB 0.97 to 1.15, above
// 0.98 to 1.16.
inline bool weights_exceed_cache(const moe_config* cfg) {
  const int64_t A = (int64_t)cfg->k * cfg->T, active = A < cfg->E ? A : cfg->E;
  const int64_t per_expert = (int64_t)(cfg->act == MOE_ACT_SWIGLU ? 3 : 2) * cfg->d_model * cfg->d_ff * (int64_t)elem_size(cfg->dtype);
  return per_expert > ((int64_t)300 << 20) / (active > 0 ? active : 1);
}

// Number of blocks of DISPATCH_BLOCK assignments the bookkeeping kernels use.
constexpr int DISPATCH_BLOCK = 256;
inline int64_t dispatch_blocks(const moe_config* cfg) {
  int64_t A = (int64_t)cfg->k * cfg->T;
  return (A + DISPATCH_BLOCK - 1) / DISPATCH_BLOCK;
}

// The grouped GEMMs hand out their tiles through one counter per XCD: the first GEMM owns ints [0,8) of a
// 16-int block, the second [8,16).  A counter must be zero when its kernel starts: the dispatch stage
// clears the first GEMM's, the first GEMM clears the second's.
constexpr int TILE_COUNTER_INTS = 16;
// Byte offset of the counters inside an MOE_WS_FFN workspace (after h[R_max, d_ff]).
size_t ffn_counter_offset(const moe_config* cfg);

// Stage launchers (arguments already validated).
bool expert_gemv_combine_one_token_applies(const moe_config* cfg);
int32_t launch_expert_gemv_combine_one_token(const moe_config* cfg, const void* h, const void* w2, const void* bias,
                                             const int32_t* offsets, const int32_t* a2r, const float* topk_w,
                                             const void* residual, void* yd, void* out, const int64_t* eoff, hipStream_t s);
bool expert_gemv_ranked_applies(const moe_config* cfg);
int32_t launch_rank_one_token(const moe_config* cfg, const double* part, int slices, const float* b_router, int32_t* topk_idx, float* topk_w,
                              int32_t* counts, int32_t* offsets, int32_t* a2r, int32_t* r2a, int32_t* clear8, hipStream_t s);
int32_t launch_expert_gemv_ranked(const moe_config* cfg, const void* x, const double* part, int slices, const float* b_router, const void* wa,
                                  const void* wb, const void* bias, void* h, const int64_t* eoff, int32_t* topk_idx, float* topk_w,
                                  int32_t* counts, int32_t* offsets, int32_t* a2r, int32_t* r2a, int32_t* clear8, hipStream_t s);
int gate_parts_one_token(const moe_config* cfg, const float* w_router, size_t scratch_bytes);
int32_t launch_gate_parts_one_token(const moe_config* cfg, const void* x, const float* w_router, double* part, size_t scratch_bytes, hipStream_t s);
bool gate_dispatch_one_token_applies(const moe_config* cfg, const float* w_router);
int32_t launch_gate_dispatch_one_token(const moe_config* cfg, const void* x, const float* w_router, const float* b_router,
                                       int32_t* topk_idx, float* topk_w, int32_t* counts, int32_t* offsets, int32_t* a2r,
                                       int32_t* r2a, int32_t* clear8, hipStream_t s);
bool gate_dispatch_slices_applies(const moe_config* cfg, const float* w_router, size_t scratch_bytes);
int32_t launch_gate_dispatch_slices(const moe_config* cfg, const void* x, const float* w_router, const float* b_router, int32_t* topk_idx,
                                    float* topk_w, int32_t* counts, int32_t* offsets, int32_t* a2r, int32_t* r2a, int32_t* clear8,
                                    void* scratch, size_t scratch_bytes, hipStream_t s);
int32_t launch_gate(const moe_config* cfg, const void* x, const float* w_router, const float* b_router,
                    int32_t* topk_idx, float* topk_w, float* probs, hipStream_t s);
// the same on the pre-split router when w carries one (moe_weights.w_router_packed) and it applies
int32_t launch_gate_of(const moe_config* cfg, const moe_weights* w, const void* x, int32_t* topk_idx, float* topk_w, float* probs,
                       hipStream_t s);
// clear8 (nullable): eight ints set to zero on the way (the first GEMM's tile counters).
int32_t launch_dispatch(const moe_config* cfg, const void* x, const int32_t* topk_idx, int32_t* counts,
                        int32_t* offsets, int32_t* a2r, int32_t* r2a, void* xd, void* ws, int32_t* clear8,
                        hipStream_t s);
// row_map (nullable): row_to_assign; xd is then x itself and the rows are gathered on the fly (float32: and stored in xd_out).
// tile_counters: the 16-int block above (bf16 only; the fp32 kernels ignore it).
int32_t launch_gemm1(const moe_config* cfg, const moe_weights* w, const void* xd, const int32_t* offsets,
                     void* h, const int32_t* row_map, int32_t* tile_counters, hipStream_t s, void* xd_out = nullptr);
bool gemm1_can_gather(const moe_config* cfg);
int32_t launch_gemm2(const moe_config* cfg, const moe_weights* w, const void* h, const int32_t* offsets,
                     void* yd, int32_t* tile_counters, hipStream_t s);
// k = 1: the second GEMM writes out[t] = residual[t] + topk_w[t] * FFN row for every token that kept its
// expert.  The others (residual[t], or zero) are written by launch_fill_dropped where the capacity can drop (a2r NULL), and
// by the same kernel where only tokens with NaN logits have no row (a2r = assign_to_row): a launch of its own costs a step of few
// tokens 2 to 3 us.  Together they replace launch_gemm2 + launch_combine and, in bf16, the dispatched-order output yd.  float32
// kernels store yd as well and write the dropped tokens themselves (a2r always).
bool gemm2_can_combine(const moe_config* cfg);
int32_t launch_gemm2_combine(const moe_config* cfg, const moe_weights* w, const void* h, const int32_t* offsets,
                             const int32_t* r2a, const float* topk_w, const void* residual, void* out,
                             const int32_t* a2r, int32_t* tile_counters, hipStream_t s, void* yd);
int32_t launch_fill_dropped(const moe_config* cfg, const int32_t* a2r, const void* residual, void* out, hipStream_t s);
int32_t launch_combine(const moe_config* cfg, const void* yd, const int32_t* a2r, const float* topk_w,
                       const void* residual, void* out, hipStream_t s);
int32_t check_weights(const moe_config* cfg, const moe_weights* w);

}  // namespace moesys
