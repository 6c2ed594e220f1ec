// Steps of one wavefront that several kernels share.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace moesys {

// Workgroup barrier for data exchanged through LDS: waits for this wavefront's LDS operations only; global loads and stores
// stay in flight.  (__syncthreads also waits for those: for results just stored, a microsecond at the end of a kernel that lasts
// ten, and for loads that are wanted a step later.)
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// An expert index as the routing tables take it: anything outside 0 .. E-1 is dropped (-1).  The gate's ranking yields such an
// index for a token that has fewer than k logits that compare at all (NaN).
__device__ __forceinline__ int valid_expert(int e, int E) { return (unsigned)e < (unsigned)E ? e : -1; }

// This lane's place among the assignments of its expert e (a valid_expert), in lane order behind the cnt[e] that came before;
// cnt (LDS, the wavefront's own, cleared by the caller) counts them on.  One ballot per bit of the index leaves every lane the
// lanes that agree with it in all bits.  A lane without an expert (-1) is nobody's neighbour, and its result means nothing.
__device__ __forceinline__ int place_in_expert(int e, int E, int* cnt, int lane) {
  unsigned long long same = __ballot(e >= 0);
  for (int bit = 1; bit < E; bit <<= 1) {
    const bool one = (e & bit) != 0;
    const unsigned long long with = __ballot(one);
    same &= one ? with : ~with;
  }
  const int rank = __popcll(same & ((1ull << lane) - 1ull));
  const int before = e >= 0 ? cnt[e] : 0;
  asm volatile("" ::: "memory");  // (a wavefront's LDS operations execute in order)
  if (e >= 0 && rank == 0) cnt[e] = before + __popcll(same);
  asm volatile("" ::: "memory");
  return before + rank;
}

// k = 1, combine in the second product's kernel, no capacity that drops: a token may still have no row (NaN logits).  Its
// output row, which no tile writes, is its residual or zero.  a2r: row of every token (NULL: the caller writes such rows
// itself); kept = offsets[E], rows there are.  The workgroups share the tokens; with a row for everyone this is one comparison.
template <int WAVES, typename X>
__device__ __forceinline__ void fill_rowless_tokens(const int32_t* __restrict__ a2r, int kept, int T, int N, const X* residual, X* out) {
  constexpr int V = 16 / sizeof(X);
  if (!a2r || kept == T || residual == out) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int first = ((int)(blockIdx.y * gridDim.x + blockIdx.x)) * WAVES + wave, step = (int)(gridDim.x * gridDim.y) * WAVES;
  for (int t = first; t < T; t += step)
    if (a2r[t] < 0)
      for (int v = lane; v < N / V; v += 64)
        reinterpret_cast<uint4*>(out)[(size_t)t * (N / V) + v] =
            residual ? reinterpret_cast<const uint4*>(residual)[(size_t)t * (N / V) + v] : uint4{0u, 0u, 0u, 0u};
}

}  // namespace moesys
