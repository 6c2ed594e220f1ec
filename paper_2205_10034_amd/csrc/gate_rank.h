// Softmax and top-k of a token by a group of eight lanes, for the kernels that rank.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace moesys {

// A lane's partner inside its group of eight consecutive lanes, for the three steps of a reduction over the group:
// steps 0 and 1 swap lanes inside a quad (lane ^ 1, lane ^ 2), step 2 mirrors the eight lanes (lane i with 7 - i,
// which lies in the other quad).  Data-parallel-primitive moves on the vector ALU: a few clocks each, where a
// general lane permutation goes through the LDS crossbar (a hundred clocks, and a reduction is a chain of them).
template <int STEP>
__device__ __forceinline__ int group8_partner(int v) {
  constexpr int ctrl = STEP == 0 ? 0xB1 /* quad_perm 1,0,3,2 */ : STEP == 1 ? 0x4E /* quad_perm 2,3,0,1 */ : 0x141 /* row_half_mirror */;
  return __builtin_amdgcn_update_dpp(0, v, ctrl, 0xF, 0xF, true);
}
template <int STEP>
__device__ __forceinline__ float group8_partner(float v) { return __int_as_float(group8_partner<STEP>(__float_as_int(v))); }
template <int STEP>
__device__ __forceinline__ double group8_partner(double v) {
  return __hiloint2double(group8_partner<STEP>(__double2hiint(v)), group8_partner<STEP>(__double2loint(v)));
}
__device__ __forceinline__ float quad_mirror(float v) {  // quad_perm 3,2,1,0
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x1B, 0xF, 0xF, true));
}
// f(step) for the three steps, unrolled
template <typename F>
__device__ __forceinline__ void group8_steps(F&& f) {
  f(std::integral_constant<int, 0>{});
  f(std::integral_constant<int, 1>{});
  f(std::integral_constant<int, 2>{});
}

// Softmax (fp32) + top-k of one token by a group of 8 adjacent lanes.  Lane `sub` of the group holds the
// float64 logits of experts sub, sub+8, ... (NPL of them, -inf beyond E).  k+1 rounds of group-wide
// arg-max (ties -> lower expert) pick the experts in rank order; the extra round only measures the gap
// to the first expert NOT selected.  Returns true (to every lane of the group) if two neighbours among
// those k+1 logits are closer than `margin`.
// MARGIN = false (logits that are exact): no extra round, returns false.
// WAVE_ORDER (E <= 64): the exponentials are added in the order of a butterfly over a wavefront with one expert per lane, so that the
// weights carry the bits of the kernel that ranks up to 16 tokens that way.
template <int NPL, bool MARGIN = true, bool WAVE_ORDER = false>
__device__ __forceinline__ bool finalize_group(double (&z)[NPL], int sub, int E, int k, int renorm, float margin,
                                               int32_t* __restrict__ idx_out, float* __restrict__ w_out,
                                               float* __restrict__ probs_out, bool mark_close = false) {
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < NPL; ++i) mx = fmaxf(mx, (float)z[i]);
  group8_steps([&](auto st) { mx = fmaxf(mx, group8_partner<decltype(st)::value>(mx)); });
  float ex[NPL], sum = 0.f;
#pragma unroll
  for (int i = 0; i < NPL; ++i) {
    ex[i] = (sub + 8 * i) < E ? expf((float)z[i] - mx) : 0.f;
    sum += ex[i];
  }
  // (the same pairs in the same order in every lane of the group: all eight hold the same sum, bit for bit)
  if constexpr (WAVE_ORDER) {
    static_assert(NPL <= 8, "a lane of the wavefront has one expert");
    float t[NPL];
#pragma unroll
    for (int i = 0; i < NPL; ++i) t[i] = ex[i];
#pragma unroll
    for (int w = NPL / 2; w >= 1; w /= 2)  // lanes 32, 16 and 8 apart
#pragma unroll
      for (int i = 0; i < w; ++i) t[i] += t[i + w];
    sum = t[0];
    sum += quad_mirror(group8_partner<2>(sum));  // 4 (7 - i, then 3 - i inside the quad), 2 and 1 apart
    sum += group8_partner<1>(sum);
    sum += group8_partner<0>(sum);
  } else {
    group8_steps([&](auto st) { sum += group8_partner<decltype(st)::value>(sum); });
  }
#pragma unroll
  for (int i = 0; i < NPL; ++i) {
    ex[i] = ex[i] / sum;
    if (probs_out && (sub + 8 * i) < E) probs_out[sub + 8 * i] = ex[i];
  }
  float my_w = 0.f, wsum = 0.f;
  int my_idx = 0;
  double prev = INFINITY;
  bool close = false;
  for (int r = 0; r < (MARGIN ? k + 1 : k); ++r) {
    double bz = -INFINITY;
    int be = 0x7fffffff;
    float bp = 0.f;
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
      const int e = sub + 8 * i;
      if (e < E && (z[i] > bz || (z[i] == bz && e < be))) { bz = z[i]; be = e; bp = ex[i]; }
    }
    group8_steps([&](auto st) {
      constexpr int S = decltype(st)::value;
      const double oz = group8_partner<S>(bz);
      const int oe = group8_partner<S>(be);
      const float op = group8_partner<S>(bp);
      if (oz > bz || (oz == bz && oe < be)) { bz = oz; be = oe; bp = op; }
    });
#pragma unroll
    for (int i = 0; i < NPL; ++i)
      if (sub + 8 * i == be) z[i] = NAN;  // retire the winner (every lane of the group agrees on be): no comparison picks it again
    if (r < k) {
      if (sub == r) { my_idx = be; my_w = bp; }
      wsum += bp;
    }
    if (MARGIN && r > 0) close |= (float)(prev - bz) < margin;
    prev = bz;
  }
  if (sub < k) {
    idx_out[sub] = my_idx;
    float w = renorm ? my_w / wsum : my_w;
    // mark_close: a token within the margin carries the sign bit on its first weight (a probability, never
    // negative otherwise) until the kernel that recomputes such tokens has replaced its results
    if (mark_close && close && sub == 0) w = __uint_as_float(__float_as_uint(w) | 0x80000000u);
    w_out[sub] = w;
  }
  return close;
}

// The same by a whole wavefront for up to 64 experts, lane e holding expert e's logit (-inf beyond E): the steps of a reduction
// over the lanes are moves on the vector ALU.  The j-th selection is returned in lane j < k, with its weight.
template <int CTRL, int ROWS, typename T>
__device__ __forceinline__ T wave_step(T v, T other) {  // `other` where the step has no source lane
  if constexpr (sizeof(T) == 8)
    return __hiloint2double(__builtin_amdgcn_update_dpp(__double2hiint(other), __double2hiint(v), CTRL, ROWS, 0xF, false),
                            __builtin_amdgcn_update_dpp(__double2loint(other), __double2loint(v), CTRL, ROWS, 0xF, false));
  else
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(other), __float_as_int(v), CTRL, ROWS, 0xF, false));
}
template <typename T, typename F>
__device__ __forceinline__ T wave_reduce(T v, T neutral, F&& f) {  // valid in lane 63 (f: any order gives the same)
  v = f(v, wave_step<0x111, 0xF>(v, neutral));  // row_shr 1, 2, 4, 8: the last lane of a row of 16 has the row's result
  v = f(v, wave_step<0x112, 0xF>(v, neutral));
  v = f(v, wave_step<0x114, 0xF>(v, neutral));
  v = f(v, wave_step<0x118, 0xF>(v, neutral));
  v = f(v, wave_step<0x142, 0xA>(v, neutral));  // row_bcast 15 into rows 1 and 3, then 31 into rows 2 and 3
  return f(v, wave_step<0x143, 0xC>(v, neutral));
}
// Sum over the lanes by a butterfly, 32, 16, 8, 4, 2 and 1 lanes apart: the bits of the same steps through __shfl_xor, in every lane.
__device__ __forceinline__ float wave_sum(float v) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  uint32_t u = __float_as_uint(v);
  const u32x2 a = __builtin_amdgcn_permlane32_swap(u, u, false, false);  // lanes 0..31 twice, lanes 32..63 twice
  u = __float_as_uint(__uint_as_float(a.x) + __uint_as_float(a.y));
  const u32x2 b = __builtin_amdgcn_permlane16_swap(u, u, false, false);  // rows of 16: the even ones twice, the odd ones twice
  v = __uint_as_float(b.x) + __uint_as_float(b.y);
  auto step = [&](auto ctrl) { v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xF, 0xF, true)); };
  step(std::integral_constant<int, 0x128>{});  // row_ror 8
  step(std::integral_constant<int, 0x124>{});  // row_ror 4: lanes 8 apart agree, so this is 4 apart
  step(std::integral_constant<int, 0x4E>{});   // quad_perm 2,3,0,1
  step(std::integral_constant<int, 0xB1>{});   // quad_perm 1,0,3,2
  return v;
}
__device__ __forceinline__ int rank_wave(double z, int lane, int E, int k, int renorm, float& weight) {
  float ex = 0.f, sum = 1.f, wsel = 0.f, wsum = 0.f;
  int isel = 0;
  for (int j = 0; j < k; ++j) {
    const double m = wave_reduce(z, -(double)INFINITY, [](double a, double b) { return b > a || a != a ? b : a; });
    const double best = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(m), 63), __builtin_amdgcn_readlane(__double2loint(m), 63));
    if (j == 0) {
      ex = lane < E ? expf((float)z - (float)best) : 0.f;
      sum = wave_sum(ex);
    }
    const unsigned long long at = __ballot(lane < E && z == best);  // ties: the lower expert; nothing that compares (NaN): none
    const int e = at ? __builtin_ctzll(at) : 0x7fffffff;
    const float p = at ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ex), e & 63)) / sum : 0.f;
    if (lane == e) z = NAN;  // retired: no comparison picks it again
    if (lane == j) { isel = e; wsel = p; }
    wsum += p;
  }
  weight = renorm ? wsel / wsum : wsel;
  return isel;
}

}  // namespace moesys
