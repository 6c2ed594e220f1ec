// Tiles of the expert products whose workgroups are not persistent: row tiles of every expert x feature tiles, counted and
// found on the device from expert_offsets.
#pragma once
#include "moesys_internal.h"

namespace moesys {

// Upper bound of the workgroups (the device counts the real tiles), a multiple of the eight XCDs.
inline int64_t row_tile_grid(const moe_config* cfg, int tile_rows, int n_tiles) {
  int64_t mt = max_rows(cfg) / tile_rows + cfg->E;  // every expert may end in one partial tile
  const int64_t C = moe_capacity(cfg);
  if (C != MOE_DROPLESS && (int64_t)cfg->E * ((C + tile_rows - 1) / tile_rows) < mt) mt = (int64_t)cfg->E * ((C + tile_rows - 1) / tile_rows);
  return (mt * n_tiles + 7) / 8 * 8;
}

struct RowTile { int expert, row0, rows, nt, tiles; };  // first dispatched row, valid rows, feature tile, row tiles of the expert

// Tile of workgroup blockIdx.x, false if there is none.  Tiles are numbered expert by expert, feature tile by feature
// tile, row tiles innermost, and every XCD (workgroup b runs on XCD b mod 8) takes one contiguous eighth: the row tiles
// that share a weight tile, and the feature tiles that share the rows, meet in one L2.  Every wavefront finds its tile
// by itself (lane l looks at the experts 4l .. 4l+3), so no barrier is spent on it.  An expert has the fewest tiles of at most TM rows.
// SHIFT: where the eighths' weights (weight_bytes a tile) lie a multiple of 16 MB apart, XCD x starts its eighth SHIFT x tiles further on and
// comes round, so that the XCDs do not meet on the same memory channels.
template <int TM, int UNIT = 0, int SHIFT = 0>
__device__ __forceinline__ bool find_row_tile(const int32_t* __restrict__ offsets, int E, int n_tiles, RowTile& t, uint32_t weight_bytes = 0) {
  const int lane = threadIdx.x & 63;
  static_assert(MOE_MAX_EXPERTS == 256, "four experts per lane");
  int cnt[4], sum = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int e = 4 * lane + j;
    cnt[j] = e < E ? (offsets[e + 1] - offsets[e] + TM - 1) / TM : 0;
    sum += cnt[j];
  }
  int incl = sum;
  for (int m = 1; 4 * m <= E; m <<= 1) {
    const int up = __shfl_up(incl, m, 64);
    incl += lane >= m ? up : 0;
  }
  // (the first E / 4 + 1 lanes have met; the later ones hold no expert)
  const int total = __builtin_amdgcn_readlane(incl, min((E + 3) / 4, 64) - 1) * n_tiles;
  const int chunk = (total + 7) / 8, i = blockIdx.x / 8, xcd = blockIdx.x % 8;
  if (i >= chunk) return false;
  int at = i;
  if (SHIFT && (uint32_t)chunk * weight_bytes % (16u << 20) == 0) at = (i + SHIFT * xcd) % chunk;
  const int id = xcd * chunk + at;
  if (id >= total) return false;
  int p = incl - sum, e = -1, base = 0, tiles = 1;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (4 * lane + j < E && id >= p * n_tiles && id < (p + cnt[j]) * n_tiles) { e = 4 * lane + j; base = p; tiles = cnt[j]; }
    p += cnt[j];
  }
  const int src = __builtin_ctzll(__ballot(e >= 0));  // (exactly one lane has it)
  e = __builtin_amdgcn_readlane(e, src);
  base = __builtin_amdgcn_readlane(base, src);
  tiles = __builtin_amdgcn_readlane(tiles, src);
  const int r = id - base * n_tiles, nt = r / tiles, m = r - nt * tiles;
  t.expert = e;
  const int n = offsets[e + 1] - offsets[e];
  // (UNIT: the rows dealt out evenly in whole units; TM is a multiple, so no tile comes out larger and none empty)
  const int per = UNIT ? ((n + tiles - 1) / tiles + UNIT - 1) / (UNIT ? UNIT : 1) * UNIT : TM;
  t.row0 = offsets[e] + m * per;
  t.rows = min(per, n - m * per);
  t.nt = nt;
  t.tiles = tiles;
  return true;
}

}  // namespace moesys
