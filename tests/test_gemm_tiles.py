"""The rules that pick a kernel and tile for a bf16 product (csrc/gemm_tiles.h), checked without a GPU: the header is plain C++, the program
below walks them over products of every kind."""
import os
import subprocess

import pytest

import test_gpu_small_tiles
import test_gpu_wide_tiles

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_18191_amd", "csrc")

WALK = r"""
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "gemm_tiles.h"
using namespace tsd;

struct Tile { int rows, cols, least_k; };
Tile of(DirectTile t) {  // rows and columns of a tile, the shortest contraction its ring of stages takes
  switch (t) {
    case kTile64: return {64, 64, 256};
    case kTile128x64: return {128, 64, 192};
    case kTile128: return {128, 128, 192};
    case kTile128x256: return {128, 256, 128};
    case kTile256x128: return {256, 128, 256};
    case kTile256: return {256, 256, 192};
    case kTileRuns: return {64, 64, 2048};
    default: return {0, 1, 0};
  }
}

// A tile that the launchers hold an instance of and that the product fits.
bool fits(int amode, int epi, DirectTile t, int M, int N, int K, int hd, int map_rows) {
  if (t == kTileNone) return true;
  const Tile s = of(t);
  if (!has_direct_kernel(amode, epi, t) || N % s.cols || K % 64 || K < s.least_k || M < 1) return false;
  if (t == kTileRuns && (!split_runs(K) || (long)((M + 63) / 64) * (N / 64) > kRunTiles)) return false;
  // a rotary pair of 32-column blocks per wavefront; wavefronts of 64 x 128 hold head_dim 64 only
  if (epi == EP_QKV && hd != 64 && (t == kTile256 || t == kTile128x256)) return false;
  return !map_rows || s.rows == map_rows;
}

int main(int argc, char** argv) {
  if (argc == 6) {  // amode epi M N K: the tile
    int v[5];
    for (int i = 0; i < 5; ++i) v[i] = atoi(argv[i + 1]);
    printf("%d\n", (int)direct_tile(v[0], v[1], v[2], v[3], v[4], 0, 0, false));
    return 0;
  }
  const int kinds[5][2] = {{A_ACT, EP_STORE}, {A_ACT, EP_RESID}, {A_NORM, EP_STORE}, {A_NORM, EP_GELU}, {A_NORM, EP_QKV}};
  long seen[5] = {0, 0, 0, 0, 0}, bad = 0, grouped = 0;
  for (int kind = 0; kind < 5; ++kind)
    for (int M = 1; M <= 40000; M += 1 + M / 17)
      for (int N = 16; N <= 4608; N += 16)
        for (int K : {8, 64, 128, 192, 256, 320, 384, 512, 520, 768, 1024, 1088, 1536, 2048, 2112, 3072, 4096})
          for (int hd : {16, 32, 64}) {
            if ((kind == 4 && N % (3 * hd)) || (kind != 4 && hd != 64)) continue;
            for (int runs = 0; runs < 2; ++runs) {
              const DirectTile t = direct_tile(kinds[kind][0], kinds[kind][1], M, N, K, hd, 0, runs);
              seen[kind] += t != kTileNone;
              bad += !fits(kinds[kind][0], kinds[kind][1], t, M, N, K, hd, 0);
            }
          }
  for (int slots = 1; slots <= 40000; slots += 1 + slots / 17)
    for (int D = 64; D <= 1024; D += 64)
      for (int F = 32; F <= 4096; F += 32)
        for (int E : {1, 2, 3, 4, 8, 16})
          for (int no_wide = 0; no_wide < 2; ++no_wide) {
            const int bm = routed_row_tile(TSD_BF16, slots, D, F, E, no_wide);
            const DirectTile up = no_wide ? kTileNone : direct_tile(A_NORM, EP_GELU, slots, F, D, 0, bm, false);
            const DirectTile down = no_wide ? kTileNone : direct_tile(A_ACT, EP_STORE, slots, D, F, 0, bm, false);
            bad += !fits(A_NORM, EP_GELU, up, slots, F, D, 0, bm) || !fits(A_ACT, EP_STORE, down, slots, D, F, 0, bm);
            // what the register-staged kernels are left with: maps of 64 or 128 rows, long contractions of activations of 64 only
            bad += up == kTileNone && bm > 128;
            bad += down == kTileNone && (bm > 128 || (bm == 128 && F >= kQuarterK));
            grouped += bm == 256;
          }
  printf("%ld %ld %ld %ld %ld %ld %ld\n", bad, grouped, seen[0], seen[1], seen[2], seen[3], seen[4]);
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("tiles")
    src, exe = tmp / "walk.cpp", tmp / "walk"
    src.write_text(WALK)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O2", "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True)
    return lambda *args: [int(x) for x in subprocess.run([str(exe), *map(str, args)], check=True, capture_output=True, text=True).stdout.split()]


def test_every_tile_the_rules_return_has_a_kernel_that_takes_the_product(walk):
    bad, grouped, *seen = walk()
    assert bad == 0 and grouped > 0 and min(seen) > 0, (bad, grouped, seen)


@pytest.mark.parametrize("M,N,K,variant,tile", test_gpu_wide_tiles.PRODUCTS + test_gpu_small_tiles.PRODUCTS)
def test_products_of_the_gpu_tests_take_the_tile_they_are_there_for(walk, M, N, K, variant, tile):
    amode, epi = {0: (2, 0), 1: (1, 0), 2: (2, 1), 3: (1, 2)}[variant]
    assert walk(amode, epi, M, N, K) == [tile]
