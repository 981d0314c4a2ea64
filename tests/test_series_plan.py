"""Index rules of the passes that take a series per workgroup (csrc/series_plan.h), checked without a GPU: the header is plain C++."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_18191_amd", "csrc")

# Pages up to the last one of the largest handle there can be (2^20 series, 64 pages each), every width, head size and page size: the
# token's first element against the layout [page][keys, values][head][token][column], counted in 128 bits, and inside a pool that size.
WALK = r"""
#include <cstdio>
#include <initializer_list>
#include "series_plan.h"
using namespace tsd;
int main() {
  long seen = 0, large = 0, wrong = 0, outside = 0;
  for (int D : {32, 64, 128})
    for (int HD : {16, 32, 64})
      for (int PT = 1; PT <= 64 && HD <= D; PT *= 2)
        for (long pages = 1; pages <= 1L << 26; pages = pages * 3 / 2 + 1)
          for (int at : {0, PT - 1}) {
            const int H = D / HD, page = (int)(pages - 1);
            const __int128 want = ((((__int128)page * 2 + 0) * H + 0) * PT + at) * HD;
            const long got = kv_token(page, at, H, PT, HD), last = got + (2L * H - 1) * PT * HD + HD - 1;
            ++seen;
            large += want >= (__int128)1 << 31;
            wrong += got != want;
            outside += got < 0 || last >= pages * 2 * PT * D;
          }
  printf("%ld %ld %ld %ld\n", seen, large, wrong, outside);
}
"""


def test_cache_offsets_of_large_batches(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    seen, large, wrong, outside = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert seen > 3000 and large > 100 and (wrong, outside) == (0, 0)
