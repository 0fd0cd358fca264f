// Arguments of the tiled GEMM kernels (vt_gemm.hip, vt_gemm_tile.hip): up to 8 products of one grouped
// launch, cut into tiles that form one list over all groups.
#pragma once

#include "vt_gemm_common.h"

namespace vt {
namespace gemm {

constexpr int kMaxGroups = 8;
constexpr int kGroupRows = 8;      // tile rows walked together (L2 reuse of the B panel)

struct GemmGroup {
  const char* a;
  const char* b;
  char* c;
  AxisMap<5> a_row;
  AxisMap<3> a_col, b_row, b_col;
  int32_t M, tile_begin, tiles_m;
  int32_t k64;   // a K step of 64 never leaves the innermost K digit of A or of B: the step's offset is uniform
  int32_t b_kmajor;   // B's contiguous axis is K (all groups of a launch agree)
};

// (NG = groups there is room for: the arguments are copied with every launch and read through the
// scalar cache before a workgroup knows its tile)
struct GemmSizes {
  int32_t n_groups, N, K, tiles_n, total_tiles, chunk, c_f32, pad;
};
template <int NG>
struct GemmGroups {
  GemmGroup g[NG];
};
template <int NG>
struct GemmParamsT : GemmGroups<NG>, GemmSizes {};
typedef GemmParamsT<kMaxGroups> GemmParams;

// Output written through a map (producer-side store, Sec. 4.2): columns [col_lo, col_hi) of C
// live in one physical tensor, element (m, n) at base + 2 * (row(m) + col(n - col_lo)).
struct OutPiece {
  char* base;
  int32_t col_lo, col_hi;
  AxisMap<3> row, col;
};
struct OutMap {
  OutPiece p[4];
  int32_t n, pad;
};
struct NoMap {};

// Which tile workgroup `wg` takes: each compute die (own L2; workgroups are dealt to them in turn)
// works on a contiguous band of the list, walked in groups of kGroupRows tile rows.  False: none.
template <int NG>
__device__ __forceinline__ bool pick_tile(const GemmParamsT<NG>& P, int wg, int* group, int* tm, int* tn) {
  const int slot = wg >> 3;
  const int idx = (wg & 7) * P.chunk + slot;
  if (slot >= P.chunk || idx >= P.total_tiles) return false;
  int gi = 0;
#pragma unroll
  for (int i = 1; i < NG; ++i)
    if (i < P.n_groups && idx >= P.g[i].tile_begin) gi = i;
  const int local = idx - P.g[gi].tile_begin;
  const int width = kGroupRows * P.tiles_n;
  const int first_m = (local / width) * kGroupRows;
  const int gsz = min(P.g[gi].tiles_m - first_m, kGroupRows);
  *group = gi;
  *tm = first_m + (local % width) % gsz;
  *tn = (local % width) / gsz;
  return true;
}

// Cuts the groups (M, N filled in) into tiles of bm x bn.
inline void set_tiles(GemmParams* P, int bm, int bn) {
  P->tiles_n = (P->N + bn - 1) / bn;
  int tiles = 0;
  for (int i = 0; i < P->n_groups; ++i) {
    P->g[i].tiles_m = (P->g[i].M + bm - 1) / bm;
    P->g[i].tile_begin = tiles;
    tiles += P->g[i].tiles_m * P->tiles_n;
  }
  P->total_tiles = tiles;
  P->chunk = (tiles + 7) / 8;
}

}  // namespace gemm
}  // namespace vt
