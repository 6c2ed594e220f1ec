// Grouped weight-gradient GEMM of the expert FFN's backward pass:
//
//   C_e[n1, n2] = sum over the rows r of expert e of A[r, n1] * B[r, n2]        (fp32 output)
//
// e.g. dW2_e = d_y_e^T h_e and dW1_e = d_u_e^T xd_e for OUTPUT_MAJOR weights.  The paper's system is a
// training system (Section 3.2) but gives no kernel; this is the chain rule on the expert FFN of the
// forward pass.  The contraction runs over an expert's rows, the SLOW index of both row-major operands,
// and its length differs per expert.
//
// CDNA4 mapping.  One workgroup per tile of one expert's C: 4 wavefronts (1 x 4, each 128 x 64) per 128 x 256, two such
// workgroups per CU; 8 (2 x 4) per 256 x 256 for long sums, 4 (2 x 2, each 64 x 64) per 128 x 128 for few tiles.  It walks the
// expert's rows 32 at a time.  Both operand chunks [32 rows x tile columns] go from global memory straight
// into LDS as they are (buffer_load ... lds, 16 bytes per lane; rows past the expert's end read as zero
// through the buffer descriptor, so the ragged length needs no padding), three stages deep.  The MFMA
// operand fragments need 8 consecutive contraction indices per lane, i.e. a COLUMN of the LDS tile: they
// are read with gfx950's transposing LDS read (ds_read_b64_tr_b16: within 16 lanes, lane i supplies a
// chunk of four 16-bit values M[i][0..3] and lane L receives M[(L mod 16)/4 + 4j][L mod 4]); with lane i
// supplying row r0 + i/4, column chunk i mod 4, lane L receives rows r0..r0+3 of column n0 + L mod 16, so
// two reads make one fragment.  The 16-byte slot index of a row is XORed with 4*(row mod 4), which lets
// the two 16-lane groups of a 32-lane pass hit all 64 banks once.
// The first MFMA operand is the n2 side, so that a lane ends up with runs of four consecutive n2 of one n1.
// Stores.  At a thousand rows per expert the gradient is as many bytes as a third of the product's time.  A wavefront's
// results go through LDS (the stages are free by then) and leave as whole 128-byte lines, past the caches: the gradient
// is not read again by this kernel, and written through L2 it drives out the operand slabs that the XCD's workgroups share.
// Two workgroups per CU let one store while the other multiplies.  Measured on MI355X, 16 experts of 1024 rows, 4096 x
// 1024 float32 (us): 256 x 256 tiles, 16 bytes per lane and row 159; the same as whole lines 153; past the caches too
// 149; 128 x 256 tiles 135 (1.02 PFLOP/s; without the whole lines 159-172; past the caches without them 185).  At 256 rows
// 79 -> 60, bf16 58 -> 45; 8 experts of 1024 rows, 11264 x 2048 bf16 375 -> 332; 64 of 128, 2048 x 4096 bf16 366 -> 238.
// At every size: an optimizer that reads the gradient at once and finds it in no cache pays for it.  Ordinary / non-temporal over 250
// random products, three sets in turn, alone and with an update p += a g right behind: up to 64 MB of gradient 1.05 and 1.00, 64 to
// 128 MB 1.08 and 0.95, above 1.15 and 1.02.  In a training step the other gradients come between, more than the caches hold.
// Tile order.  The 8 XCDs have an L2 each, and the hardware deals workgroups out to them round robin.  A tile
// streams a slab of A and one of B; tiles of one expert with the same n1 (n2) tile share the A (B) slab.  The tiles of
// an expert are numbered in blocks of BY x BX, the experts one after the other, and units of `unit` consecutive tiles are
// dealt out to the XCDs in turn: 32, or evenly fewer, so that no XCD gets more than a unit's rounding more than another.
// (Units of what an XCD runs at once, 64 or 96 tiles, are no faster with even routing and put a hot expert of 64 tiles on one XCD: 8
// experts, 2048 x 512, half of 5600 rows on one: 38.7 us.)  (Blocks dealt out whole, partial ones too, met on the same XCDs where their number per expert
// has a factor in common with eight: 64 experts of 81 rows, 768 x 2560 bf16, 96 against 70 us; over 150 random shapes the
// units gain 4.5 %.)
// Column sums of A per expert (the bias gradients: db2_e = sum_r d_y[r, :], db1_e = sum_r d_u[r, :]) come from
// the same fragments: the workgroups of the first n2 tile multiply one n1 fragment per wavefront and K-step
// by a fragment of ones (one more MFMA on top of eight), which leaves the column's sum in every element of
// that accumulator.  No extra pass over A.
#include <type_traits>
#include "moesys_internal.h"

namespace moesys {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int WG_N = 256;        // multiple that N1 and N2 must be of
constexpr int WG_KS = 32;        // rows per K-step
constexpr int CU_PER_XCD = 32;
// Tile of TN1 x TN2: W1 x W2 wavefronts, each N1B blocks of 32 n1 columns x two of n2
template <int TN1, int TN2, int N1B_>
struct WgShape {
  static constexpr int N1B = N1B_, W1 = TN1 / (32 * N1B), W2 = TN2 / 64, WAVES = W1 * W2;
  static constexpr int ROW_A = TN1 * 2, ROW_B = TN2 * 2;                       // bytes of one LDS row
  static constexpr int CHUNK_A = WG_KS * ROW_A, CHUNK_B = WG_KS * ROW_B;       // one operand chunk
  static constexpr int LOADS_A = CHUNK_A / 1024 / WAVES, LOADS_B = CHUNK_B / 1024 / WAVES;  // wave-wide 1 KB loads per wavefront and stage
};
constexpr int wg_wait_vm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0f70; }  // at most n vector memory operations in flight

#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t wg_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
#endif

template <bool COLSUM, bool OUT_BF16, int TN1, int TN2, int N1B>
__global__ __launch_bounds__((WgShape<TN1, TN2, N1B>::WAVES * 64), 2) void grouped_wgrad_kernel(
    const uint16_t* __restrict__ a,       // [R, N1]
    const uint16_t* __restrict__ b,       // [R, N2]
    const int32_t* __restrict__ offsets,  // [E+1]
    void* __restrict__ c_out,             // [E, N1, N2] float32, or bfloat16 (OUT_BF16: one rounding of the fp32 sums)
    float* __restrict__ a_colsum,         // COLSUM: [E, N1]
    int N1, int N2, int E, int BY, int BX, int unit) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef WgShape<TN1, TN2, N1B> S;
  constexpr int WG_WAVES = S::WAVES, W2 = S::W2, CHUNK_A = S::CHUNK_A, STAGE = S::CHUNK_A + S::CHUNK_B;
  // one array per stage: the compiler can then tell the stage being filled from the one being read
  __shared__ __attribute__((aligned(1024))) unsigned char s0[STAGE];
  __shared__ __attribute__((aligned(1024))) unsigned char s1[STAGE];
  __shared__ __attribute__((aligned(1024))) unsigned char s2[STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w1 = wave / W2, w2 = wave % W2;  // this wavefront: n1 columns [32*N1B*w1, +32*N1B), n2 columns [64*w2, +64)
  // workgroup -> (expert, n1 tile, n2 tile): see "Tile order" above
  const int n1t = N1 / TN1, n2t = N2 / TN2;
  const int slot = blockIdx.x / 8;                       // position in this XCD's sequence of workgroups
  const int id = ((slot / unit) * 8 + (int)(blockIdx.x % 8)) * unit + slot % unit;  // units are dealt out to the XCDs in turn
  if (id >= E * n1t * n2t) return;
  const int e = id / (n1t * n2t), in_e = id - e * (n1t * n2t);
  const int band = in_e / (BY * n2t), in_band = in_e - band * (BY * n2t), band_rows = min(BY, n1t - band * BY);
  const int cblk = in_band / (band_rows * BX), in_blk = in_band - cblk * (band_rows * BX), cols = min(BX, n2t - cblk * BX);
  const int ty = band * BY + in_blk / cols, tx = cblk * BX + in_blk % cols;
  const int row0 = offsets[e], rows = offsets[e + 1] - row0;
  const int t1 = ty * TN1, t2 = tx * TN2;
  const size_t c_tile = ((size_t)e * N1 + t1) * N2 + t2;  // element offset of this tile in c
  const int KT = (rows + WG_KS - 1) / WG_KS;

  // ---- direct-to-LDS loads: one instruction = 1 KB = 2 or 4 rows of a chunk in slots of 16 bytes; a lane's physical slot
  // holds the logical slot ^ key(row), key = 4 * (row mod 4) (the rows of a lane's loads are a multiple of four apart).
  constexpr int SLOTS_A = S::ROW_A / 16, SLOTS_B = S::ROW_B / 16, STEP_A = WG_WAVES * 64 / SLOTS_A, STEP_B = WG_WAVES * 64 / SLOTS_B;
  static_assert(STEP_A % 4 == 0 && STEP_B % 4 == 0 && STEP_A * S::LOADS_A == WG_KS && STEP_B * S::LOADS_B == WG_KS, "whole stages, one key per lane");
  const uint32_t a_pitch = (uint32_t)N1 * 2u, b_pitch = (uint32_t)N2 * 2u;
  auto lane_offset = [&](int slots, int pitch, int first) {
    const int row = (64 / slots) * wave + lane / slots;
    return row * pitch + first * 2 + ((lane % slots) ^ (4 * (row & 3))) * 16;
  };
  const int a_voff = lane_offset(SLOTS_A, (int)a_pitch, t1), b_voff = lane_offset(SLOTS_B, (int)b_pitch, t2);
  const uint16_t* a_base = a + (size_t)row0 * N1;
  const uint16_t* b_base = b + (size_t)row0 * N2;
  const uint32_t a_bytes = (uint32_t)rows * a_pitch, b_bytes = (uint32_t)rows * b_pitch;
  auto issue = [&](int kt, unsigned char* stage) {
    const bool live = kt < KT;
    const __amdgpu_buffer_rsrc_t ra = wg_rsrc(a_base, live ? a_bytes : 0u), rb = wg_rsrc(b_base, live ? b_bytes : 0u);
    const int r0 = kt * WG_KS;
#pragma unroll
    for (int i = 0; i < S::LOADS_A; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (__attribute__((address_space(3))) void*)(stage + (i * WG_WAVES + wave) * 1024), 16,
                                               a_voff, (r0 + STEP_A * i) * (int)a_pitch, 0, 0);
#pragma unroll
    for (int i = 0; i < S::LOADS_B; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (__attribute__((address_space(3))) void*)(stage + CHUNK_A + (i * WG_WAVES + wave) * 1024), 16,
                                               b_voff, (r0 + STEP_B * i) * (int)b_pitch, 0, 0);
  };

  // ---- transposing fragment reads: lane L, 16-lane group g = L / 16, i = L mod 16 supplies row
  // 8*(g/2) + 4*h + i/4 (h = 0, 1: the two halves of its 8 contraction indices), columns 16*(g%2) + 4*(i%4)..+3
  // of the 32-column block; key(row) = 4 * ((i/4) mod 4) for every row it supplies.
  const int g = lane >> 4, li = lane & 15;
  const int fr_row = 8 * (g >> 1) + (li >> 2);                 // + 4*h + 16*ks
  const int fr_col = 16 * (g & 1) + 4 * (li & 3);              // column inside the 32-column block
  const int fr_key = 4 * ((li >> 2) & 3);
  auto frag_addr = [&](int col0) {  // byte offset of this lane's chunk for the block starting at column col0, row part excluded
    const int col = col0 + fr_col;
    return (((col >> 3) ^ fr_key) << 4) + ((col >> 2) & 1) * 8;
  };
  int n1_addr[N1B], n2_addr[2];
#pragma unroll
  for (int i = 0; i < N1B; ++i) n1_addr[i] = frag_addr(32 * N1B * w1 + 32 * i) + fr_row * S::ROW_A;
#pragma unroll
  for (int j = 0; j < 2; ++j) n2_addr[j] = frag_addr(64 * w2 + 32 * j) + fr_row * S::ROW_B;
  auto read_frag = [&](const unsigned char* chunk, int addr, int ks, auto row_tag) {
    constexpr int ROW = decltype(row_tag)::value;
    const unsigned char* p = chunk + addr + ks * 16 * ROW;
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)p);
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(p + 4 * ROW));
    bf16x8 f;
    const bf16x4 l4 = __builtin_bit_cast(bf16x4, lo), h4 = __builtin_bit_cast(bf16x4, hi);
#pragma unroll
    for (int q = 0; q < 4; ++q) { f[q] = l4[q]; f[4 + q] = h4[q]; }
    return f;
  };

  f32x16 acc[N1B][2];
#pragma unroll
  for (int i = 0; i < N1B; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // column sums: wavefront (w1, w2) of the first n2 tile's workgroups sums the n1 block i = w2 of its columns
  const bool do_colsum = COLSUM && tx == 0;
  f32x16 acc_sum;
  bf16x8 ones;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc_sum[v] = 0.f;
#pragma unroll
  for (int v = 0; v < 8; ++v) ones[v] = (__bf16)1.0f;

  auto compute = [&](const unsigned char* stage) {
#pragma unroll
    for (int ks = 0; ks < WG_KS / 16; ++ks) {
      bf16x8 f1[N1B], f2[2];
#pragma unroll
      for (int i = 0; i < N1B; ++i) f1[i] = read_frag(stage, n1_addr[i], ks, std::integral_constant<int, S::ROW_A>{});
#pragma unroll
      for (int j = 0; j < 2; ++j) f2[j] = read_frag(stage + CHUNK_A, n2_addr[j], ks, std::integral_constant<int, S::ROW_B>{});
#pragma unroll
      for (int i = 0; i < N1B; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f2[j], f1[i], acc[i][j], 0, 0, 0);
      if constexpr (COLSUM) {
        if (do_colsum) {
          bf16x8 mine = f1[0];
#pragma unroll
          for (int i = 1; i < N1B; ++i) mine = w2 == i ? f1[i] : mine;
          acc_sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, mine, acc_sum, 0, 0, 0);
        }
      }
    }
  };

  // ---- K loop, three stages: the loads of K-steps kt+1 and kt+2 stay in flight while K-step kt is
  // multiplied (past the last K-step the loads are zero-length, so the count in flight is the same)
  issue(0, s0);
  issue(1, s1);
  issue(2, s2);
  // After a stage's barrier other wavefronts' loads overwrite it, and the zero-length ones store their zeros without a way
  // to memory first: every wavefront's fragment reads have come back before it arrives (lgkmcnt(0) only).
  constexpr int READS_DONE = 0xc07f;
  constexpr int TWO_STAGES = wg_wait_vm(2 * (S::LOADS_A + S::LOADS_B));
  for (int kt = 0; kt < KT; kt += 3) {
    __builtin_amdgcn_s_waitcnt(TWO_STAGES);  // this wavefront's share of the stage has landed
    __builtin_amdgcn_s_barrier();
    compute(s0);
    __builtin_amdgcn_s_waitcnt(READS_DONE);
    __builtin_amdgcn_s_barrier();
    issue(kt + 3, s0);
    if (kt + 1 < KT) {
      __builtin_amdgcn_s_waitcnt(TWO_STAGES);
      __builtin_amdgcn_s_barrier();
      compute(s1);
      __builtin_amdgcn_s_waitcnt(READS_DONE);
      __builtin_amdgcn_s_barrier();
    }
    issue(kt + 4, s1);
    if (kt + 2 < KT) {
      __builtin_amdgcn_s_waitcnt(TWO_STAGES);
      __builtin_amdgcn_s_barrier();
      compute(s2);
      __builtin_amdgcn_s_waitcnt(READS_DONE);
      __builtin_amdgcn_s_barrier();
    }
    issue(kt + 5, s2);
  }
  __builtin_amdgcn_s_waitcnt(0x0070);  // the zero-length tail loads retire
  __syncthreads();                     // ... every wavefront's: the stages are free

  // ---- epilogue: lane holds n1 = lane & 31 of each n1 block and n2 = 8*q + 4*(lane >> 5) + 0..3 of each n2 block.  A
  // wavefront's 32 rows of n1 x 64 columns of n2 go through its own piece of the stages, 16-byte slots XORed with the row,
  // and leave as whole 256-byte (bf16: 128-byte) row segments.
  constexpr int ES = OUT_BF16 ? 2 : 4, SEG = 64 * ES, SLOTS = SEG / 16, BUF = 32 * SEG, PER = STAGE / BUF;
  static_assert(2 * PER >= WG_WAVES, "every wavefront has a piece of the first two stages");
  unsigned char* const buf = wave < PER ? s0 + wave * BUF : s1 + (wave - PER) * BUF;
  const int o1 = lane & 31, hi = lane >> 5;
#pragma unroll
  for (int i = 0; i < N1B; ++i) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if constexpr (OUT_BF16) {
#pragma unroll
        for (int q = 0; q < 4; q += 2) {
          auto pk = [&](int qq, int r) {
            const bf16x2 h = __builtin_convertvector(f32x2{acc[i][j][4 * qq + r], acc[i][j][4 * qq + r + 1]}, bf16x2);
            return __builtin_bit_cast(uint32_t, h);
          };
          const u32x2 sx = __builtin_amdgcn_permlane32_swap(pk(q, 0), pk(q + 1, 0), false, false);
          const u32x2 sy = __builtin_amdgcn_permlane32_swap(pk(q, 2), pk(q + 1, 2), false, false);
          *reinterpret_cast<u32x4*>(buf + o1 * SEG + (((4 * j + q + hi) ^ (o1 & (SLOTS - 1))) << 4)) = u32x4{sx.x, sy.x, sx.y, sy.y};
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 v = {acc[i][j][4 * q + 0], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          *reinterpret_cast<f32x4*>(buf + o1 * SEG + (((8 * j + 2 * q + hi) ^ (o1 & (SLOTS - 1))) << 4)) = v;
        }
      }
    }
    // (one wavefront's LDS operations execute in order; this keeps the compiler from moving reads of other lanes' slots)
    asm volatile("" ::: "memory");
    constexpr int RPI = 64 / SLOTS;  // rows per wave-wide store
    const int row = lane / SLOTS, slot_ = lane % SLOTS;
    u32x4 v[32 / RPI];
#pragma unroll
    for (int m = 0; m < 32 / RPI; ++m)
      v[m] = *reinterpret_cast<const u32x4*>(buf + (m * RPI + row) * SEG + ((slot_ ^ ((m * RPI + row) & (SLOTS - 1))) << 4));
    asm volatile("" ::: "memory");
#pragma unroll
    for (int m = 0; m < 32 / RPI; ++m) {
      u32x4* dst = reinterpret_cast<u32x4*>((char*)c_out + (c_tile + (size_t)(32 * N1B * w1 + 32 * i + m * RPI + row) * N2 + 64 * w2) * ES + slot_ * 16);
      __builtin_nontemporal_store(v[m], dst);
    }
  }
  if constexpr (COLSUM) {
    // every element of acc_sum in lane l (and l + 32) is the sum of column 32*N1B*w1 + 32*w2 + (l & 31)
    if (do_colsum && lane < 32) a_colsum[(size_t)e * N1 + t1 + 32 * N1B * w1 + 32 * w2 + lane] = acc_sum[0];
  }
#endif
}

// Tiles of the XCD that gets most of them when blocks of BY x BX tiles are dealt out whole.  The kernel deals out even units, so
// this is no load of its XCDs; it measures how raggedly an expert's tiles divide into blocks, and thus how many slabs of operands
// the tiles that run together on an XCD share.
int64_t busiest_xcd(int E, int n1t, int n2t, int BX, int BY) {
  int64_t load[8] = {}, most = 0;
  int x = 0;
  for (int e = 0; e < E; ++e)
    for (int y = 0; y < n1t; y += BY)
      for (int c = 0; c < n2t; c += BX, x = (x + 1) % 8) load[x] += (int64_t)(n1t - y < BY ? n1t - y : BY) * (n2t - c < BX ? n2t - c : BX);
  for (int64_t l : load) most = l > most ? l : most;
  return most;
}

// Edge along n2: 256 (3 transposing LDS reads per 2 MFMAs against 4 per 2 for 128 x 128) unless 256 x 256 tiles leave a quarter
// of their rounds of 256 CUs empty and do not divide more raggedly when they are smaller.  The line (62 small tiles of an XCD
// against its 64 for whole rounds of 32 large ones) was drawn when blocks were dealt out whole and is no model of the present
// order.  Over 500 random products, a quarter under Zipf routing, the best of the three tiles takes 0.973 of its time, one tile
// always 0.99 (128 x 128), 1.13 (128 x 256) and 1.31 (256 x 256); most of what it gives away is under Zipf routing, where a hot
// expert's sums are long (64 experts, 512 x 512, 699 / 365 with 128 x 128).  Of 250 products three are slower than with the tiles and order
// before these, by up to 10 %.  Measured on MI355X (us, 128 x 256 / 128 x 128): 4 experts of
// 1840 rows, 2048 x 512 f32 33 / 23; 4 of 708, 1024 x 1536 f32 19 / 17; 4 of 2525, 1792 x 1280 bf16 64 / 57.  Past that line either may
// win by a tenth: 4 experts of 230 rows, 2048 x 2304 f32 26 / 21; 8 of 1004, 4096 x 1024 74 / 81; 32 of 1653, 1024 x 5376 560 / 646.
// Edge along n1 beside 256: 128, two workgroups per CU that cover each other's start and stores.  256 where the operands are
// read most: from 1400 rows on, or with more operand bytes than the 256 MB last-level cache holds, unless the larger tiles lose
// more to their last round than the 4 % they gain.  (us, 128 x 256 / 256 x 256): 16 experts of 2048 rows, 4096 x 1024 f32 271 / 260;
// of 1024 135 / 149; 16 of 4026, 512 x 1792 124 / 114; 64 of 350, 8192 x 1536 f32 (436 MB) 1097 / 987; 64 of 300, 4096 x 2048 (236
// MB) 483 / 533; 16 of 2557, 2304 x 1024 (2.25 rounds) 178 / 198.
// Columns of tiles per block (BX): eight, or as wide as the gradient's rows, up to 32, with few rows per expert, where the
// stores bound the product.
struct WgTiles { int TN, TN1, BX; };  // edges along n2 and n1, columns of tiles per block
WgTiles wgrad_tiles(int E, int N1, int N2, int c_dtype, int64_t rows_per_expert) {
  auto busiest = [&](int tn, int bx) { return busiest_xcd(E, N1 / tn, N2 / tn, bx, 32 / bx); };
  auto columns = [&](int tn) {
    const int n2t = N2 / tn, eight = n2t < 8 ? n2t : 8, all = n2t < 32 ? n2t : 32;
    if (tn != 256 || n2t <= 8 || rows_per_expert > 160) return eight;
    if (n2t < 16) return all;
    if (c_dtype == MOE_BF16 && n2t % 32 == 0 && (int64_t)E * N1 * N2 * 2 >= ((int64_t)1 << 30)) return all;
    return rows_per_expert <= 32 && busiest(256, all) <= busiest(256, 8) ? all : eight;
  };
  const int64_t tiles = (int64_t)E * (N1 / 256) * (N2 / 256), rounds = (tiles + 255) / 256;
  int TN = 256;
  if (tiles <= 512 && 4 * tiles < 3 * 256 * rounds) {
    const int64_t large = (busiest(256, columns(256)) + 31) / 32, small = busiest(128, columns(128));
    if (small * 62 < large * 64 * 100) TN = 128;
  }
  const int64_t half_rounds = (2 * tiles + 255) / 256;
  const bool long_sums = rows_per_expert >= 1400 || (int64_t)E * rows_per_expert * (N1 + N2) * 2 > ((int64_t)256 << 20);
  const bool whole = TN == 256 && long_sums && 2 * rounds * 96 <= half_rounds * 100;
  return {TN, whole ? 256 : 128, columns(TN)};
}

}  // namespace

int32_t launch_wgrad_bf16(const uint16_t* a, const uint16_t* b, const int32_t* offsets, void* c, int c_dtype, float* a_colsum, int E,
                          int N1, int N2, int64_t max_rows_per_expert, int64_t rows_per_expert, hipStream_t s) {
  if (c_dtype != MOE_F32 && c_dtype != MOE_BF16) return fail(MOE_ERR_INVALID_ARG, "weight gradient: output type must be MOE_F32 or MOE_BF16");
  if (N1 % WG_N || N2 % WG_N) return fail(MOE_ERR_UNSUPPORTED, "weight gradient: N1=%d and N2=%d must be multiples of %d", N1, N2, WG_N);
  const int64_t widest = N1 > N2 ? N1 : N2;
  if ((max_rows_per_expert + WG_KS) * widest * 2 >= ((int64_t)1 << 31))
    return fail(MOE_ERR_UNSUPPORTED, "weight gradient: an expert's operand block exceeds 2 GiB");
  const bool h = c_dtype == MOE_BF16;
  const WgTiles t = wgrad_tiles(E, N1, N2, c_dtype, rows_per_expert);
  const int BX = t.BX, n1t = N1 / t.TN1, n2t = N2 / t.TN;
  // blocks of 32 tiles, units of at most as many
  const int BY = CU_PER_XCD / BX;
  const int64_t tiles = (int64_t)E * n1t * n2t, units = (tiles + 8 * CU_PER_XCD - 1) / (8 * CU_PER_XCD);  // (of one XCD)
  const int unit = (int)((tiles + 8 * units - 1) / (8 * units));
  const int64_t wgs = 8 * units * unit;
  if (wgs > INT32_MAX) return fail(MOE_ERR_UNSUPPORTED, "weight gradient: too many tiles");
  auto run = [&](auto t1, auto t2, auto nb) {
    constexpr int A = decltype(t1)::value, B = decltype(t2)::value, C = decltype(nb)::value;
    auto kern = a_colsum ? (h ? grouped_wgrad_kernel<true, true, A, B, C> : grouped_wgrad_kernel<true, false, A, B, C>)
                         : (h ? grouped_wgrad_kernel<false, true, A, B, C> : grouped_wgrad_kernel<false, false, A, B, C>);
    hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(WgShape<A, B, C>::WAVES * 64), 0, s, a, b, offsets, c, a_colsum, N1, N2, E, BY, BX, unit);
  };
  using std::integral_constant;
  if (t.TN == 128) run(integral_constant<int, 128>{}, integral_constant<int, 128>{}, integral_constant<int, 2>{});
  else if (t.TN1 == 128) run(integral_constant<int, 128>{}, integral_constant<int, 256>{}, integral_constant<int, 4>{});
  else run(integral_constant<int, 256>{}, integral_constant<int, 256>{}, integral_constant<int, 4>{});
  return check_hip(hipGetLastError(), "weight gradient launch");
}

}  // namespace moesys

using namespace moesys;

extern "C" int32_t moe_expert_wgrad(const void* a, const void* b, const int32_t* expert_offsets, void* c, int32_t c_dtype,
                                    float* a_column_sums, int32_t E, int32_t N1, int32_t N2, int64_t max_rows_per_expert,
                                    void* stream) {
  if (!a || !b || !expert_offsets || !c) return fail(MOE_ERR_INVALID_ARG, "moe_expert_wgrad: NULL argument");
  if (E < 1 || E > MOE_MAX_EXPERTS || N1 < 1 || N2 < 1 || max_rows_per_expert < 0)
    return fail(MOE_ERR_INVALID_ARG, "moe_expert_wgrad: bad shape");
  return launch_wgrad_bf16((const uint16_t*)a, (const uint16_t*)b, expert_offsets, c, c_dtype, a_column_sums, E, N1, N2,
                           max_rows_per_expert, max_rows_per_expert, (hipStream_t)stream);
}

// Tile edge along n2 and width of a block of tiles (TN * 100 + BX), tile edge along n1: for the tests of the rule above.  Host only; not part of the
// interface in moesys.h.
extern "C" int32_t moe_test_wgrad_tiles(int32_t E, int32_t N1, int32_t N2, int32_t c_dtype, int64_t rows_per_expert) {
  const moesys::WgTiles t = moesys::wgrad_tiles(E, N1, N2, c_dtype, rows_per_expert);
  return t.TN * 100 + t.BX;
}
extern "C" int32_t moe_test_wgrad_n1_edge(int32_t E, int32_t N1, int32_t N2, int32_t c_dtype, int64_t rows_per_expert) {
  return moesys::wgrad_tiles(E, N1, N2, c_dtype, rows_per_expert).TN1;
}
