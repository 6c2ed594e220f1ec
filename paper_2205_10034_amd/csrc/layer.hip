// moe_layer_forward: gate -> dispatch -> expert FFN -> combine on one stream with one workspace,
// and the stage timer used by the bench to attribute time per kernel group.
#include <new>
#include "moesys_internal.h"

struct moe_timer {
  hipEvent_t ev[MOE_STAGE_COUNT + 1];
  bool recorded;
};

namespace moesys {
namespace {

struct Segments {
  int32_t *topk_idx, *counts, *offsets, *a2r, *r2a, *tile_ctr;
  float* topk_w;
  void *xd, *h, *yd, *scratch;
};

// Validates what both halves of the layer need and resolves the workspace segments.
int32_t open_workspace(const char* who, const moe_config* cfg, const moe_weights* w, const void* x, void* ws,
                       size_t ws_bytes, Segments* sg) {
  int32_t st = moe_config_check(cfg);
  if (st != MOE_OK) return st;
  if (!w) return fail(MOE_ERR_INVALID_ARG, "%s: weights is NULL", who);
  if (cfg->T > 0 && !x) return fail(MOE_ERR_INVALID_ARG, "%s: x must be non-NULL", who);
  moe_ws_layout L;
  moe_workspace_layout(cfg, &L);
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < L.total)
    return fail(MOE_ERR_WORKSPACE, "%s: workspace needs %zu bytes, 256-byte aligned (got %zu)", who, L.total, ws_bytes);
  char* base = (char*)ws;
  sg->topk_idx = (int32_t*)(base + L.topk_idx);
  sg->topk_w = (float*)(base + L.topk_w);
  sg->counts = (int32_t*)(base + L.expert_counts);
  sg->offsets = (int32_t*)(base + L.expert_offsets);
  sg->a2r = (int32_t*)(base + L.assign_to_row);
  sg->r2a = (int32_t*)(base + L.row_to_assign);
  sg->xd = base + L.xd;
  sg->h = base + L.h;
  sg->yd = base + L.yd;
  sg->scratch = base + L.scratch;
  sg->tile_ctr = (int32_t*)(base + L.tile_counters);
  return MOE_OK;
}

int32_t mark(moe_timer* timer, int i, hipStream_t s) {
  if (!timer) return MOE_OK;
  return check_hip(hipEventRecord(timer->ev[i], s), "hipEventRecord");
}

size_t h_bytes(const moe_config* cfg) { return (size_t)max_rows(cfg) * cfg->d_ff * elem_size(cfg->dtype); }

// A one-token step: the gate's partial logits, then ranking and tables, inside a layer in the first product's kernel, in routing alone
// in one of their own.  The partial logits lie in yd inside a layer, whose first product reads them while it writes h, and in h in
// routing alone, which leaves yd as it is.  The same bits in both: the same sums in the same order, or, where h has room for fewer
// slices than yd, float64 sums in another order (as many slices as either holds would cost the layer: 64 experts 4096 x 512, k 2 18.7
// us with the sixteen of yd, 22.8 with the four of h).
size_t yd_bytes(const moe_config* cfg) { return (size_t)max_rows(cfg) * cfg->d_model * elem_size(cfg->dtype); }
int one_token_parts(const moe_config* cfg, const moe_weights* w, bool alone) {  // 0: not such a step, or no room
  return expert_gemv_ranked_applies(cfg) ? gate_parts_one_token(cfg, w->w_router, alone ? h_bytes(cfg) : yd_bytes(cfg)) : 0;
}

// Inside a layer or, alone, in moe_layer_route: a one-token step's partial logits, ranked by a kernel of their own or by the first
// product; slices and one ranking workgroup; one kernel for gate and tables of a token; the gate's kernels and the dispatch's.
// Routing alone in two launches where one kernel (gate_few_kernel) could serve, for the layer's bits.  Measured on MI355X, routers of
// 8 x 512 to 64 x 1920, one kernel / two (us): 6.5 to 9 / 3.1 + 2.4 on the card; a call and a wait for its tables, as an expert pool
// makes it, 24.3 to 27.4 / 23.7 to 24.7, then the experts and a wait 63.7 / 60.1 (16 x 2048 x 2816); calls one after the other without a
// look at the tables, which moe_layer_forward serves, are bound by the host's launches: 9.8 / 12.1 to 13.4.
enum Routing { ROUTE_RANK_ONE, ROUTE_RANKED_PRODUCT, ROUTE_SLICES, ROUTE_ONE_TOKEN, ROUTE_GATE };
Routing pick_routing(const moe_config* cfg, const moe_weights* w, bool alone) {
  if (one_token_parts(cfg, w, true) > 0) return !alone && one_token_parts(cfg, w, false) > 0 ? ROUTE_RANKED_PRODUCT : ROUTE_RANK_ONE;
  if (!gemm1_can_gather(cfg)) return ROUTE_GATE;
  if (gate_dispatch_slices_applies(cfg, w->w_router, h_bytes(cfg))) return ROUTE_SLICES;
  return gate_dispatch_one_token_applies(cfg, w->w_router) ? ROUTE_ONE_TOKEN : ROUTE_GATE;
}

// gate -> dispatch bookkeeping (and, on the fp32 path, the dispatched copy, unless the first product makes it: rows = false)
int32_t route_impl(const char* who, const moe_config* cfg, const moe_weights* w, const void* x, void* ws,
                   size_t ws_bytes, hipStream_t s, moe_timer* timer, bool rows = true) {
  Segments sg;
  int32_t st = open_workspace(who, cfg, w, x, ws, ws_bytes, &sg);
  if (st != MOE_OK) return st;
  if (!w->w_router) return fail(MOE_ERR_INVALID_ARG, "%s: w_router is NULL", who);
  if ((st = mark(timer, 0, s)) != MOE_OK) return st;
  const bool gather = gemm1_can_gather(cfg);
  const Routing how = pick_routing(cfg, w, true);
  if (how == ROUTE_RANK_ONE) {
    if ((st = launch_gate_parts_one_token(cfg, x, w->w_router, (double*)sg.h, h_bytes(cfg), s)) != MOE_OK) return st;
    if ((st = launch_rank_one_token(cfg, (const double*)sg.h, one_token_parts(cfg, w, true), w->b_router, sg.topk_idx, sg.topk_w,
                                    sg.counts, sg.offsets, sg.a2r, sg.r2a, sg.tile_ctr, s)) != MOE_OK)
      return st;
    if ((st = mark(timer, 1, s)) != MOE_OK) return st;
    return mark(timer, 2, s);
  }
  // few tokens: the gate runs on many compute units and writes the dispatch tables as well (the partial logits go
  // where the first product will write)
  if (how == ROUTE_SLICES) {
    if ((st = launch_gate_dispatch_slices(cfg, x, w->w_router, w->b_router, sg.topk_idx, sg.topk_w, sg.counts, sg.offsets, sg.a2r,
                                          sg.r2a, sg.tile_ctr, sg.h, h_bytes(cfg), s)) != MOE_OK)
      return st;
    if ((st = mark(timer, 1, s)) != MOE_OK) return st;
    return mark(timer, 2, s);
  }
  if (how == ROUTE_ONE_TOKEN) {
    // a step of one token: the gate's kernel writes the dispatch tables as well
    if ((st = launch_gate_dispatch_one_token(cfg, x, w->w_router, w->b_router, sg.topk_idx, sg.topk_w, sg.counts, sg.offsets,
                                             sg.a2r, sg.r2a, sg.tile_ctr, s)) != MOE_OK)
      return st;
    if ((st = mark(timer, 1, s)) != MOE_OK) return st;
    return mark(timer, 2, s);
  }
  if ((st = launch_gate_of(cfg, w, x, sg.topk_idx, sg.topk_w, nullptr, s)) != MOE_OK) return st;
  if ((st = mark(timer, 1, s)) != MOE_OK) return st;
  // bf16: the first GEMM gathers its rows from x through row_to_assign, so no dispatched copy is made
  if ((st = launch_dispatch(cfg, x, sg.topk_idx, sg.counts, sg.offsets, sg.a2r, sg.r2a, gather || !rows ? nullptr : sg.xd,
                            sg.scratch, sg.tile_ctr, s)) != MOE_OK)
    return st;
  return mark(timer, 2, s);
}

int32_t route_and_first_product(const char* who, const moe_config* cfg, const moe_weights* w, const void* x, void* ws, size_t ws_bytes,
                                hipStream_t s, moe_timer* timer) {
  Segments sg;
  int32_t st = open_workspace(who, cfg, w, x, ws, ws_bytes, &sg);
  if (st != MOE_OK) return st;
  const bool sw = cfg->act == MOE_ACT_SWIGLU;
  double* part = (double*)sg.yd;
  if ((st = mark(timer, 0, s)) != MOE_OK) return st;
  if ((st = launch_gate_parts_one_token(cfg, x, w->w_router, part, yd_bytes(cfg), s)) != MOE_OK) return st;
  if ((st = mark(timer, 1, s)) != MOE_OK) return st;
  if ((st = mark(timer, 2, s)) != MOE_OK) return st;
  return launch_expert_gemv_ranked(cfg, x, part, one_token_parts(cfg, w, false), w->b_router, sw ? w->w_gate_proj : w->w1,
                                   sw ? w->w_up : nullptr, sw ? nullptr : w->b1, sg.h, w->expert_elem_offset, sg.topk_idx, sg.topk_w,
                                   sg.counts, sg.offsets, sg.a2r, sg.r2a, sg.tile_ctr, s);
}

// expert FFN -> combine, from the routing tables in the workspace (after_first: the first product has run; rows = false: float32,
// the dispatched rows are still to be made, from x)
int32_t experts_impl(const char* who, const moe_config* cfg, const moe_weights* w, const void* x, const void* residual,
                     void* out, void* ws, size_t ws_bytes, hipStream_t s, moe_timer* timer, bool after_first = false,
                     bool rows = true) {
  Segments sg;
  int32_t st = open_workspace(who, cfg, w, x, ws, ws_bytes, &sg);
  if (st != MOE_OK) return st;
  if ((st = check_weights(cfg, w)) != MOE_OK) return st;
  if (cfg->T > 0 && !out) return fail(MOE_ERR_INVALID_ARG, "%s: out must be non-NULL", who);
  if (out == x && residual != x) return fail(MOE_ERR_INVALID_ARG, "%s: out aliases x", who);
  const bool gather = gemm1_can_gather(cfg);
  const bool direct = gather || !rows;  // the first product reads x
  if (!after_first && (st = launch_gemm1(cfg, w, direct ? x : sg.xd, sg.offsets, sg.h, direct ? sg.r2a : nullptr, sg.tile_ctr, s,
                                         rows ? nullptr : sg.xd)) != MOE_OK)
    return st;
  if ((st = mark(timer, 3, s)) != MOE_OK) return st;
  if (cfg->k == 1) {
    // one expert per token: the second GEMM scales each row by its gate weight, adds the residual and writes
    // it to its token's place; what is left of the combine stage are the rows of dropped tokens.  An expert gets at most T
    // rows: unless C is smaller only tokens with NaN logits have none, and the second GEMM writes those as well
    const int64_t C = moe_capacity(cfg);
    // (float32: its kernels write those in any case)
    const bool drops = cfg->dtype == MOE_BF16 && C != MOE_DROPLESS && C < cfg->T;
    if ((st = launch_gemm2_combine(cfg, w, sg.h, sg.offsets, sg.r2a, sg.topk_w, residual, out, drops ? nullptr : sg.a2r, sg.tile_ctr, s, sg.yd)) != MOE_OK)
      return st;
    if ((st = mark(timer, 4, s)) != MOE_OK) return st;
    if (drops)
      if ((st = launch_fill_dropped(cfg, sg.a2r, residual, out, s)) != MOE_OK) return st;
  } else if (expert_gemv_combine_one_token_applies(cfg)) {
    // a step of one token with several experts: the second product and the combine in one kernel (same yd, same out)
    const bool sw = cfg->act == MOE_ACT_SWIGLU;
    if ((st = launch_expert_gemv_combine_one_token(cfg, sg.h, sw ? w->w_down : w->w2, sw ? nullptr : w->b2, sg.offsets, sg.a2r,
                                                   sg.topk_w, residual, sg.yd, out, w->expert_elem_offset, s)) != MOE_OK)
      return st;
    if ((st = mark(timer, 4, s)) != MOE_OK) return st;
  } else {
    if ((st = launch_gemm2(cfg, w, sg.h, sg.offsets, sg.yd, sg.tile_ctr, s)) != MOE_OK) return st;
    if ((st = mark(timer, 4, s)) != MOE_OK) return st;
    if ((st = launch_combine(cfg, sg.yd, sg.a2r, sg.topk_w, residual, out, s)) != MOE_OK) return st;
  }
  if ((st = mark(timer, 5, s)) != MOE_OK) return st;
  if (timer) timer->recorded = true;
  return MOE_OK;
}

// float32 inside a layer: the first product gathers its rows from x and its tiles store the dispatched copy on their way, which saves a
// launch, but the more a tile has to copy for the features it computes, the longer it holds its compute unit.  MI355X, layers of 16 MB of
// dispatched rows and more, copied by a kernel of its own / by the first product: below 768 features 0.98 over 295 (111 of them more than
// 2 % slower; 8 experts, 4399 tokens, k 2, 1984 x 128: 183 / 215 us), from 768 on 1.002 over 216 (2).  8 to 16 MB 1.006 and 1.003, less 1.064 and
// 1.026.
bool first_product_copies(const moe_config* cfg) {
  return cfg->dtype == MOE_F32 && ((size_t)max_rows(cfg) * cfg->d_model * 4 < ((size_t)16 << 20) || cfg->d_ff >= 768);
}

int32_t layer_impl(const moe_config* cfg, const moe_weights* w, const void* x, const void* residual, void* out,
                   void* ws, size_t ws_bytes, hipStream_t s, moe_timer* timer) {
  // everything is validated before anything is launched
  int32_t st = moe_config_check(cfg);
  if (st != MOE_OK) return st;
  if ((st = check_weights(cfg, w)) != MOE_OK) return st;
  if (cfg->T > 0 && (!x || !out)) return fail(MOE_ERR_INVALID_ARG, "moe_layer_forward: x and out must be non-NULL");
  if (out == x && residual != x) return fail(MOE_ERR_INVALID_ARG, "moe_layer_forward: out aliases x");
  if (w->w_router && pick_routing(cfg, w, false) == ROUTE_RANKED_PRODUCT) {
    if ((st = route_and_first_product("moe_layer_forward", cfg, w, x, ws, ws_bytes, s, timer)) != MOE_OK) return st;
    return experts_impl("moe_layer_forward", cfg, w, x, residual, out, ws, ws_bytes, s, timer, true);
  }
  const bool rows = !first_product_copies(cfg);
  if ((st = route_impl("moe_layer_forward", cfg, w, x, ws, ws_bytes, s, timer, rows)) != MOE_OK) return st;
  return experts_impl("moe_layer_forward", cfg, w, x, residual, out, ws, ws_bytes, s, timer, false, rows);
}

}  // namespace
}  // namespace moesys

using namespace moesys;

extern "C" {

const char* moe_test_gate_kernel(const moe_config* cfg, int32_t packed);

int32_t moe_layer_forward(const moe_config* cfg, const moe_weights* w, const void* x, const void* residual,
                          void* out, void* ws, size_t ws_bytes, void* stream) {
  return layer_impl(cfg, w, x, residual, out, ws, ws_bytes, (hipStream_t)stream, nullptr);
}

int32_t moe_layer_route(const moe_config* cfg, const moe_weights* w, const void* x, void* ws, size_t ws_bytes,
                        void* stream) {
  return route_impl("moe_layer_route", cfg, w, x, ws, ws_bytes, (hipStream_t)stream, nullptr);
}

int32_t moe_layer_experts(const moe_config* cfg, const moe_weights* w, const void* x, const void* residual,
                          void* out, void* ws, size_t ws_bytes, void* stream) {
  return experts_impl("moe_layer_experts", cfg, w, x, residual, out, ws, ws_bytes, (hipStream_t)stream, nullptr);
}

int32_t moe_layer_forward_timed(const moe_config* cfg, const moe_weights* w, const void* x, const void* residual,
                                void* out, void* ws, size_t ws_bytes, void* stream, moe_timer* timer) {
  if (!timer) return fail(MOE_ERR_INVALID_ARG, "moe_layer_forward_timed: timer is NULL");
  return layer_impl(cfg, w, x, residual, out, ws, ws_bytes, (hipStream_t)stream, timer);
}

int32_t moe_timer_create(moe_timer** out) {
  if (!out) return fail(MOE_ERR_INVALID_ARG, "moe_timer_create: out is NULL");
  moe_timer* t = new (std::nothrow) moe_timer();
  if (!t) return fail(MOE_ERR_HIP, "moe_timer_create: out of host memory");
  t->recorded = false;
  for (int i = 0; i <= MOE_STAGE_COUNT; ++i) {
    hipError_t e = hipEventCreate(&t->ev[i]);
    if (e != hipSuccess) {
      for (int j = 0; j < i; ++j) (void)hipEventDestroy(t->ev[j]);
      delete t;
      return check_hip(e, "hipEventCreate");
    }
  }
  *out = t;
  return MOE_OK;
}

int32_t moe_timer_destroy(moe_timer* t) {
  if (!t) return MOE_OK;
  for (int i = 0; i <= MOE_STAGE_COUNT; ++i) (void)hipEventDestroy(t->ev[i]);
  delete t;
  return MOE_OK;
}

int32_t moe_timer_read(moe_timer* t, float* stage_ms) {
  if (!t || !stage_ms) return fail(MOE_ERR_INVALID_ARG, "moe_timer_read: NULL argument");
  if (!t->recorded) return fail(MOE_ERR_STATE, "moe_timer_read: no timed call recorded");
  int32_t st = check_hip(hipEventSynchronize(t->ev[MOE_STAGE_COUNT]), "hipEventSynchronize");
  if (st != MOE_OK) return st;
  for (int i = 0; i < MOE_STAGE_COUNT; ++i) {
    st = check_hip(hipEventElapsedTime(&stage_ms[i], t->ev[i], t->ev[i + 1]), "hipEventElapsedTime");
    if (st != MOE_OK) return st;
  }
  return MOE_OK;
}

// How a layer (alone = 0) or moe_layer_route (alone = 1) gets its routing tables, with or without a packed router (16-byte aligned
// weights): for the tests of the rules.  Host only; not part of the interface in moesys.h.
const char* moe_test_layer_routing(const moe_config* cfg, int32_t packed, int32_t alone) {
  if (moe_config_check(cfg) != MOE_OK) return "";
  const moe_weights w = {};
  switch (pick_routing(cfg, &w, alone != 0)) {
    case ROUTE_RANK_ONE: return "parts + ranking";
    case ROUTE_RANKED_PRODUCT: return "parts + ranking product";
    case ROUTE_SLICES: return "slices";
    case ROUTE_ONE_TOKEN: return "one token";
    case ROUTE_GATE: break;
  }
  return moe_test_gate_kernel(cfg, packed);
}

// Whether the first product of a float32 layer makes the dispatched copy: for the test of the rule.
int32_t moe_test_first_product_copies(const moe_config* cfg) { return moe_config_check(cfg) == MOE_OK && first_product_copies(cfg); }

}  // extern "C"
