"""Index rules of the passes that take a series per workgroup (csrc/series_plan.h), checked without a GPU: the header is plain C++."""
import os
import subprocess

import pytest

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


def _build(folder, source):
    src, exe = folder / "walk.cpp", folder / "walk"
    src.write_text(source)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return lambda *args: [int(x) for x in subprocess.run([str(exe), *map(str, args)], check=True, capture_output=True, text=True).stdout.split()]


def test_cache_offsets_of_large_batches(tmp_path):
    seen, large, wrong, outside = _build(tmp_path, WALK)()
    assert seen > 3000 and large > 100 and (wrong, outside) == (0, 0)


PAYS = r"""
#include <cstdio>
#include <cstdlib>
#include "series_plan.h"
int main(int, char** a) { printf("%d", tsd::series_context_pays(atoi(a[1]), atoi(a[2]), atoi(a[3]))); }
"""


@pytest.fixture(scope="module")
def pays(tmp_path_factory):
    run = _build(tmp_path_factory.mktemp("pays"), PAYS)
    return lambda *args: bool(run(*args)[0])


# Times of the launch-by-launch path over those of a workgroup per series, measured: (wider model, series, tokens).
@pytest.mark.parametrize("case", [(64, 1536, 1), (64, 2048, 3), (64, 16384, 9), (64, 64, 128), (64, 96, 112), (128, 768, 1), (128, 4096, 3),
                                  (128, 16384, 7), (128, 64, 74), (128, 96, 96), (128, 129, 101), (32, 2048, 1), (32, 32768, 12), (32, 65536, 17),
                                  (64, 1, 95), (128, 1, 63)])
def test_contexts_that_are_slower_by_a_series_per_workgroup(pays, case):
    assert not pays(*case)  # (0.16 to 0.98)


@pytest.mark.parametrize("case", [(64, 1, 1), (64, 512, 1), (64, 768, 3), (64, 1, 64), (64, 64, 65), (64, 129, 128), (64, 16384, 17), (64, 4096, 12),
                                  (128, 512, 1), (128, 1280, 7), (128, 1, 32), (128, 64, 33), (128, 129, 89), (128, 16384, 16), (32, 512, 1),
                                  (32, 16384, 16)])
def test_contexts_that_are_faster_by_a_series_per_workgroup(pays, case):
    assert pays(*case)  # (1.04 to 6.1)
