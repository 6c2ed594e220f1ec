// The table of the normal distribution function that the bf16 kernels' GELU epilogues read.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace moesys {

typedef float phi_f32x2 __attribute__((ext_vector_type(2)));

// gelu(u) = u * Phi(u).  Phi comes from a table in LDS: PHI_N entries on x_i = -PHI_RANGE + i / PHI_SCALE, filled
// once per workgroup with the exact erf, and read with linear interpolation.  An entry is the line through
// (x_i, Phi(x_i)) and (x_i+1, Phi(x_i+1)) as (intercept, slope) in u itself, so that the interpolation is one
// fused multiply-add of u (no fractional part to extract; the intercept is of order one, its rounding 1e-7).
// Interpolation error <= h^2/8 * max|Phi''| = (1/64)^2 / 8 * 0.242 = 7.4e-6, far below the
// bf16 rounding of h; outside the range Phi is 0 or 1 to 6e-16.  A table read plus ~8 ALU operations
// replaces ~50 for the library erff: the activation runs on every element of h while the matrix pipes
// wait, so its instruction count is what the GEMM1 epilogue costs.
constexpr int PHI_N = 1024;
constexpr float PHI_RANGE = 8.0f, PHI_SCALE = 64.0f;

__device__ __forceinline__ void fill_phi_table(phi_f32x2* tab) {
  for (int i = threadIdx.x; i < PHI_N; i += blockDim.x) {
    const float x0 = -PHI_RANGE + (float)i / PHI_SCALE, x1 = -PHI_RANGE + (float)(i + 1) / PHI_SCALE;
    const float p0 = 0.5f * erfcf(-x0 * 0.70710678118654752f), p1 = 0.5f * erfcf(-x1 * 0.70710678118654752f);
    // the two end cells also serve everything outside the range: constants there (Phi is 0 or 1 to 6e-16)
    const float slope = (i == 0 || i == PHI_N - 1) ? 0.f : (p1 - p0) * PHI_SCALE;
    tab[i] = phi_f32x2{p0 - slope * x0, slope};
  }
}
// LDS address of the table cell of u (entries of 8 bytes).  u is clamped into the range, scaled to bytes and added
// to 2^23 + the table's own LDS address: at that magnitude a float's unit in the last place is 1, so the sum's
// low mantissa bits ARE the rounded address, and masking the low three bits (the table is 8-byte aligned) and the
// bits above the LDS leaves the cell's address.  (Rounding to nearest instead of down moves the upper sixteenth
// of a cell to the next cell's line, read h/16 outside its cell: error f'' h^2 / 32, below the h^2 / 8 inside a
// cell.)  Three instructions (clamp, multiply-add, mask) where convert-to-integer, shift and base add took four.
constexpr float PHI_CLAMP_HI = PHI_RANGE - 1.0f / 256.0f;
typedef __attribute__((address_space(3))) const phi_f32x2* phi_lds_ptr;
// the addend of phi_cell(): 2^23 + (offset of u = 0 in bytes) + the table's LDS address
__device__ __forceinline__ float phi_addend(const phi_f32x2* tab) {
  const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)tab;
  return 8388608.0f + PHI_RANGE * PHI_SCALE * 8.0f + (float)base;  // (all integers below 2^24: exact)
}
// The read is written as table base + (address - table base): the two constants cancel in the generated code, and
// the compiler still knows which LDS object is read.  With a bare integer address it cannot tell the read from
// the LDS writes of the direct-to-LDS loads in flight (the next tile's first stages) and waits for all of them.
__device__ __forceinline__ phi_f32x2 phi_cell(float u, float addend, const phi_f32x2* tab) {
  const float c = __builtin_amdgcn_fmed3f(u, -PHI_RANGE, PHI_CLAMP_HI);
  const float tm = fmaf(c, PHI_SCALE * 8.0f, addend);
  const uint32_t addr = __float_as_uint(tm) & 0x3fff8u;  // (LDS addresses are below 2^18)
  const auto base = (__attribute__((address_space(3))) const char*)tab;
  return *(phi_lds_ptr)(base + (addr - (uint32_t)(uintptr_t)base));
}
// B values at a time, in three passes: table positions, the B table reads back to back, the
// interpolations.  (One value at a time the compiler waits for every read before it starts the next
// value, and the epilogue then runs at the latency of the LDS instead of at the rate of the vector ALU.)
template <int B>
__device__ __forceinline__ void gelu_table_n(float* u, float addend, const phi_f32x2* tab) {
  phi_f32x2 e[B];
#pragma unroll
  for (int r = 0; r < B; ++r) e[r] = phi_cell(u[r], addend, tab);
#pragma unroll
  for (int r = 0; r < B; ++r) u[r] *= fmaf(u[r], e[r].y, e[r].x);
}
}  // namespace moesys
