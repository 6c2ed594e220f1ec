// Dispatch tables of up to 1024 R assignments by one workgroup of 16 wavefronts, for the kernels that end with them.
#pragma once
#include "moesys_internal.h"
#include "wave_util.h"

namespace moesys {

// Exclusive prefix of the kept rows per expert by the first wavefront: lane l owns the experts 4l .. 4l + 3.
__device__ __forceinline__ void prefix_offsets(const int* total_s, int* off_s, int E, int C, int wave, int lane) {
  if (wave != 0) return;
  static_assert(MOE_MAX_EXPERTS == 256, "four experts per lane");
  int own[4], sum = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int e = 4 * lane + j;
    own[j] = sum;
    sum += e < E ? min(total_s[e], C) : 0;
  }
  int incl = sum;
  for (int m = 1; 4 * m <= E; m <<= 1) {  // (lanes 0 .. E / 4 meet: the last writes off_s[E])
    const int up = __shfl_up(incl, m, 64);
    incl += lane >= m ? up : 0;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int e = 4 * lane + j;
    if (e <= E) off_s[e] = incl - sum + own[j];  // (e == E: the experts before it are all there are)
  }
  if (E == MOE_MAX_EXPERTS && lane == 63) off_s[E] = incl;
}

// The workgroup's A assignments: thread (wave, lane) has those with a = (wave R + r) 64 + lane, their experts (valid_expert, -1
// past the last) in e_of.  A wavefront ranks its 64 R consecutive assignments 64 at a time against its own running counts, the
// wavefronts' counts meet in LDS.  s: nobody else may use it from the call on.
constexpr int ONE_WAVES = 16;
struct OneTables {
  int cnt[ONE_WAVES][MOE_MAX_EXPERTS];  // per wavefront: assignments of every expert, then those before the wavefront's
  int total[MOE_MAX_EXPERTS];
  int off[MOE_MAX_EXPERTS + 1];
};
template <int R>
__device__ __forceinline__ void write_tables(const int (&e_of)[R], int A, int E, int C, OneTables& s, int32_t* __restrict__ counts,
                                             int32_t* __restrict__ offsets, int32_t* __restrict__ a2r, int32_t* __restrict__ r2a) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int slot[R];
  for (int e = lane; e < E; e += 64) s.cnt[wave][e] = 0;
  asm volatile("" ::: "memory");  // (a wavefront's LDS operations execute in order)
#pragma unroll
  for (int r = 0; r < R; ++r) slot[r] = place_in_expert(e_of[r], E, s.cnt[wave], lane);
  __syncthreads();
  if (tid < E) {
    int run = 0;
#pragma unroll
    for (int w = 0; w < ONE_WAVES; ++w) {
      const int c = s.cnt[w][tid];
      s.cnt[w][tid] = run;
      run += c;
    }
    s.total[tid] = run;
  }
  __syncthreads();
  prefix_offsets(s.total, s.off, E, C, wave, lane);
  __syncthreads();
  for (int i = tid; i <= E; i += ONE_WAVES * 64) {
    offsets[i] = s.off[i];
    if (i < E) counts[i] = s.total[i];
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int a = (wave * R + r) * 64 + lane, e = e_of[r];
    if (a >= A) continue;
    int row = -1;
    if (e >= 0) {
      const int in = slot[r] + s.cnt[wave][e];
      if (in < C) row = s.off[e] + in;
    }
    a2r[a] = row;
    if (row >= 0) r2a[row] = a;
  }
}

}  // namespace moesys
