// Which kernel and tile a bf16 product takes: sizes and rules, in plain C++ so that they can be checked without a GPU
// (tests/test_gemm_tiles.py).
#pragma once
#include "tsd.h"

namespace tsd {

// ---- A-operand sources and epilogues of the fused GEMM family ------------------------------
enum AMode {
  A_TOK = 0,   // fp32 patches gathered from two per-series segments (patch embedding)
  A_NORM = 1,  // fp32 residual stream; RMSNorm applied as a per-row scale of the product
  A_ACT = 2,   // activations already in the compute dtype
  A_NORM32 = 3 // like A_NORM but reads the fp32 residual itself (output head; split hi+lo in bf16 mode)
};
enum Epi {
  EP_STORE = 0,  // x = C                       (fp32)
  EP_RESID = 1,  // x += C                      (fp32 residual stream)
  EP_GELU = 2,   // h = GELU_tanh(C)            (compute dtype)
  EP_QKV = 3,    // RoPE on q,k; q -> buffer, k,v -> paged KV cache
  EP_HEAD = 4    // mu = C, fp32, scattered to [series][token - t_skip]
};

// bf16 products of activations with K >= kQuarterK are summed in four runs of k-steps (see gemm.hip)
constexpr int kQuarterK = 1024;
// ... and, where every run is at least as long as a tile's ring, the runs can be workgroups of their own (gemm_direct64.hip)
constexpr bool split_runs(int K) { return K >= kQuarterK && K % 64 == 0 && K / 64 - 3 * ((K / 64 + 3) / 4) >= 4; }
constexpr int kRunTiles = 112;  // 64 x 64 tiles of such a product at most
// From K = 2048 on a workgroup per run is faster than any other way while all of them are resident together, two per compute unit,
// with room to spare (split workgroups of gemm.hip / a workgroup per run, us: 256x512x2048 9.9 / 7.0, 768x512x2048, 96 tiles, 10.2 / 10.0;
// 256x768x3072 13.4 / 8.8, 558x768x3072, 108, 13.7 / 12.2, 768x768x3072, 144, 13.7 / 15.6; 320x1024x4096, 80, 16.7 / 11.5, 558, 144,
// 17.0 / 17.1); shorter ones gain nothing (256x1024x1024 6.95 / 7.04).
constexpr bool takes_runs(int N, int K, int M) { return K >= 2048 && split_runs(K) && N % 64 == 0 && (long)((M + 63) / 64) * (N / 64) <= kRunTiles; }
// The tiles of the direct-to-LDS kernels (gemm_direct64.hip, gemm_wide.hip); kTileNone: the register-staged kernels (gemm.hip).
enum DirectTile { kTileNone = 0, kTile64 = 64, kTile128x64 = 127, kTile128 = 128, kTile128x256 = 129, kTile256x128 = 256, kTile256 = 257, kTileRuns = 464 };

// The instances there are: the rules below may return no other, the launchers hold no other.
constexpr bool has_direct_kernel(int amode, int epi, DirectTile tile) {
  const bool act = amode == A_ACT && (epi == EP_STORE || epi == EP_RESID), norm = amode == A_NORM && (epi == EP_STORE || epi == EP_GELU || epi == EP_QKV);
  switch (tile) {
    case kTile64: case kTile128: return act || norm;
    case kTile256x128: return act;
    case kTile256: case kTile128x64: return norm && epi != EP_STORE;
    case kTile128x256: return norm && epi == EP_QKV;
    case kTileRuns: return act && epi == EP_RESID;
    default: return false;
  }
}

// Row-tile size the launcher will use for an M x N product (the routed FFN builds its tile map for it).
inline int gemm_row_tile(int dtype, int M, int N, int force_bm) {
  if (dtype != TSD_BF16) return 64;
  if (force_bm) return force_bm;
  const long t128 = (long)((M + 127) / 128) * ((N + 127) / 128);
  // 128 x 128 tiles once there are at least 1.5 of them per CU; below that the 64 x 64 tiles, four times as many,
  // keep more of the chip busy (threshold found by timing whole passes: 192 .. 1024 tried)
  return t128 >= 384 ? 128 : 64;
}

// Which direct-to-LDS tile, if any, this product should take (kTileNone: the register-staged kernels of gemm.hip).  Every kernel
// gives the same bits, so the product's shape alone decides.  Measured over M of 256 to 16343 and models of 512, 768 and 1024
// columns, weights of 24 layers in turn; us.
// hd: of a QKV product's heads; map_rows: of a tile of a grouped product's map (0: dense); runs: there is room for the sums of a long
// contraction's runs.
inline DirectTile direct_tile(int amode, int epi, int M, int N, int K, int hd, int map_rows, bool runs) {
  if (!has_direct_kernel(amode, epi, kTile128) || (K % 64) || K < 192) return kTileNone;
  // grouped products of the routed FFN: their tile map was built for tiles of so many rows (routed_row_tile)
  if (map_rows) {
    if (map_rows == 256) return amode == A_NORM ? kTile256 : kTile256x128;
    return map_rows == 128 && N % 128 == 0 ? kTile128 : kTileNone;
  }
  auto tiles = [&](int bm, int bn) { return (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  const long t64 = tiles(64, 64), t128 = tiles(128, 128);
  // Long contractions with at most one 64 x 64 tile per compute unit are latency-bound chains of k-steps, where four groups of
  // wavefronts that stream a quarter of K each (gemm.hip) are faster: 1280x512x2048 10.2 split, 11.5 here; 512x1024x4096 17.2 / 18.9.
  const bool split = amode == A_ACT && K >= kQuarterK && t64 <= 256;
  if (split && runs && epi == EP_RESID && takes_runs(N, K, M)) return kTileRuns;
  const DirectTile narrow = !split && K >= 256 && N % 64 == 0 ? kTile64 : kTileNone;
  if (amode == A_NORM && epi != EP_STORE) {
    const bool heads64 = epi != EP_QKV || hd == 64;  // (one rotary pair of blocks per 64 columns of a wavefront)
    // 256 x 256: 14 + 20 K / 1024 us per round of one tile per compute unit, the fewest operand bytes of all; taken where its rounds
    // are four fifths full (16343x4096x1024, 4 rounds: 144 against 162 at 128 x 256 and 166 at 128 x 128; 7168x4096x1024, 1.75: 67 / 75
    // / 75; 4608x3072x1024, 0.84: 37 / 40 / 43; but 12000x3072x768, 2.2 of 3 rounds: 83 / 79 / 76)
    if (heads64 && N % 256 == 0) {
      const long t256 = tiles(256, 256), rounds = (t256 + 255) / 256;
      if (5 * t256 >= 4 * 256 * rounds) return kTile256;
      // QKV only: 7168x3072x1024 60 against 66 at 128 x 128, 16343x1536x512 41 / 44, 12000x3072x1024 98 / 100
      if (epi == EP_QKV && tiles(128, 256) >= 512) return kTile128x256;
    }
    // one 64 x 64 tile per compute unit or less: the fewest k-steps in a row (558x1536x512 6.1 against 7.0 at 128 x 64)
    if (narrow && t64 <= 256) return narrow;
    // ... two or more: 128 x 64 tiles, two or three workgroups per compute unit (64 x 64 / 128 x 64 / 128 x 128: 1280x1536x512 8.0 / 7.3 /
    // 10.9, 1000x3072x768 14.4 / 11.1 / 13.2, 1280x4096x1024 23 / 19 / 21), up to three of them.  (From 513 to 640 tiles of 128 x 128
    // they are 6 to 12 % faster alone, too, but no whole forecast moved: 0.998, 1.002, 1.002.)
    if (N % 64 == 0 && (N % 128 || tiles(128, 64) <= 768)) return kTile128x64;
    return N % 128 == 0 ? kTile128 : narrow;
  }
  if (N % 128) return narrow;
  // Two 64 x 64 tiles per compute unit or less (2000x1024x4096 29 against 37 at 128 x 128)
  if (narrow && t64 <= 512) return narrow;
  // the long contractions of activations: 256 x 128 with three stages (16343x1024x4096 131 against 142 at 128 x 128, 4608x1024x4096, 144 tiles, 57 / 63)
  if (amode == A_ACT && K >= 2048 && tiles(256, 128) >= 140) return kTile256x128;
  // up to one 128 x 128 tile per compute unit three stages (4608x768x3072, 216 tiles, 32 against 36 with two and 41 at 64 x 64;
  // 4608x768x768 12.8 / 14.1 / 14.8), beyond two workgroups with two; short contractions need some more of them
  // (12000x384x384, 282, 12.0 at 128 x 128 and 11.6 at 64 x 64)
  if (!split && (t128 >= 384 || K >= 512)) return kTile128;
  return narrow;
}

// Rows of a tile of the grouped products of a routed FFN (`slots` assignments, FFN D x F, E experts): both walk one tile map.
// 256 (256 x 256 up, 256 x 128 down, one workgroup per compute unit) where the rounds of both are four fifths full, as long as the
// experts' last tiles do not spill into another one: half a tile each on average, three quarters allowed for.  Up + down, us, 128 rows /
// 256 rows: 768 x 3072, 8 experts, 9200 slots (2 rounds, 1) 72 + 58 / 64 + 53, 25600 167 + 165 / 152 + 159; 1024 x 4096, 4 experts,
// 15360 168 + 159 / 151 + 138; but 768 x 3072, 10240 slots (3, 2) 77 + 60 / 85 + 86, 16000, a choice each, (4, 2) 112 + 108 / 120 + 103.
inline int routed_row_tile(int dtype, int slots, int D, int F, int E, bool no_wide) {
  const int bm = gemm_row_tile(dtype, slots, F, 0);
  if (bm < 128) return bm;
  const bool direct = !no_wide && D % 128 == 0 && F % 64 == 0;
  if (direct && D >= 192 && F % 256 == 0) {
    const long rows = slots / 256 + 3 * E / 4;
    auto full = [](long t) { return 5 * t >= 4 * 256 * ((t + 255) / 256); };
    if (full(rows * (F / 256)) && full(rows * (D / 128))) return 256;
  }
  // the second product is a long contraction of activations from F = kQuarterK on: of the kernels with 128-row tiles only the
  // direct-to-LDS ones take it (they keep the running sum of its four runs)
  return F >= kQuarterK && !direct ? 64 : 128;
}

}  // namespace tsd
