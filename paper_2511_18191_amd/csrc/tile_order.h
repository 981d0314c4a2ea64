// Which tile of a product a workgroup takes, shared by the tiled GEMM kernels.
#pragma once
#include "tsd_internal.h"

namespace tsd {

// Workgroups go round-robin to the 8 XCDs (each with its own L2), so workgroup w lands on XCD w % 8.  Give every XCD one contiguous run of the
// tile list, and order the list in groups of 8 tile columns walked row by row: the ~32 tiles an XCD runs at a time then form a 4 x 8
// rectangle that shares 4 row panels and 8 column panels through that L2.  False: no tile (a grid is padded to whole runs, and a replayed
// launch may be larger than the tile list: workgroups past an XCD's run must not wander into the next XCD's).
__device__ __forceinline__ bool own_tile(int tiles_m, int tiles_n, int& tm, int& tn) {
  const int n_tiles = tiles_m * tiles_n;
  const int per_xcd = (n_tiles + 7) >> 3;
  if ((int)(blockIdx.x >> 3) >= per_xcd) return false;
  const int lin = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (lin >= n_tiles) return false;
  constexpr int GW = 8;
  const int gc = lin / (GW * tiles_m), rem = lin - gc * (GW * tiles_m);
  const int gw = min(GW, tiles_n - gc * GW);
  tm = rem / gw;
  tn = gc * GW + rem - tm * gw;
  return true;
}

// Row tiles of a product: of its rows, or, in grouped mode, as many as the map holds.
template <int BM>
__device__ __forceinline__ int row_tiles(const GemmP& p, int M) {
  return p.tile_map ? reinterpret_cast<const int4*>(p.tile_map)[p.n_mtiles].x : (M + BM - 1) / BM;
}

}  // namespace tsd
