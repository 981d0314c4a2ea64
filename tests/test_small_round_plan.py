"""Index rules of the resident decode kernel (csrc/small_round_plan.h), checked without a GPU: the header is plain C++, the program
below walks the reads of every product the kernel accepts."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_18191_amd", "csrc")

READS = r"""
#include <cstdio>
#include "small_round_plan.h"
using namespace tsd;

// Every read of a product's rows (or weights): wavefront, part of its four slabs, k-step, 16-byte piece of a k-step.  All of them
// have to end inside the row, so that those of row 31 end inside the part of the exchange buffer that the stage was given.
long outside(const SmallPlan& d, long row_bytes) {
  long bad = 0;
  for (int wave = 0; wave < kSmallRoundWorkers && kSmallRoundWorkers * wave < d.used; ++wave)
    for (int part = 0; part < 4; ++part)
      for (int j = 0; j < d.per; ++j)
        for (int piece = 0; piece < 4; ++piece) {
          const long first = ((slab_read(wave, part, d.used) * d.per + j) * 32 + piece * 8) * 2L;
          bad += first < 0 || first + 16 > row_bytes;
        }
  return bad;
}

int main() {
  long products = 0, ragged = 0, bad = 0, gaps = 0, overlaps = 0;
  for (int K = 32; K <= 4096; K += 32)
    for (int N = 4; N <= 4096; N += 4)
      if (small_product_ok(K, N)) {
        const SmallPlan d = small_plan(K, N);
        ++products;
        ragged += d.used % 4 != 0;
        bad += outside(d, 2L * K);
        // the slabs that count are read where they lie
        for (int s = 0; s < d.used; ++s) gaps += slab_read(s / 4, s % 4, d.used) != s;
      }
  // the parts of a layer follow one another, rows of 32
  for (int D = 64; D <= 1024; D += 64)
    for (int F = 32; F <= 4096; F += 32) {
      const size_t width[5] = {(size_t)D, (size_t)D, (size_t)D, (size_t)D, (size_t)F};
      const int part[5] = {kIn, kQuery, kMixed, kMid, kHidden};
      for (int i = 0; i < 5; ++i) {
        const size_t end = small_part_offset(D, part[i]) + kSmallRoundRows * width[i] * 2;
        overlaps += end > (i < 4 ? small_part_offset(D, part[i + 1]) : small_slab_bytes(D, F));
      }
      overlaps += small_slab_bytes(D, F) % 128 != 0 || small_part_offset(D, kQuery) % 128 != 0;  // (no line belongs to two parts)
    }
  printf("%ld %ld %ld %ld %ld\n", products, ragged, bad, gaps, overlaps);
}
"""


def _run(tmp_path, source):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(source)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return [int(x) for x in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()]


def test_reads_stay_inside_their_part(tmp_path):
    products, ragged, bad, gaps, overlaps = _run(tmp_path, READS)
    assert products > 10000 and ragged > 1000      # products whose last worker has fewer than four slabs are among them
    assert (bad, gaps, overlaps) == (0, 0, 0)


def test_reads_of_a_full_four_slabs_would_leave_their_part(tmp_path):
    """What the rule is for: with the slab taken as it comes, the walk above finds reads outside."""
    source = READS.replace("slab_read(wave, part, d.used) * d.per", "(kSmallRoundWorkers * wave + part) * d.per")
    assert source != READS and _run(tmp_path, source)[2] > 0


def test_widths_the_kernel_takes(tmp_path):
    """As include/tsd.h states them: of the widths up to 1024 in whole heads all but 320 and 448."""
    out = _run(tmp_path, '''
#include <cstdio>
#include "small_round_plan.h"
int main() {
  for (int D = 64; D <= 1024; D += 64)
    if (!tsd::small_product_ok(D, 3 * D) || !tsd::small_product_ok(D, D)) printf("%d ", D);
}
''')
    assert out == [320, 448]


EPOCHS = r"""
#include <cstdio>
#include <initializer_list>
#include "small_round_plan.h"
using namespace tsd;
int main() {
  // launches in which no series is active, one after the other, past two turns of the counter, then one that waits: no stage of it may
  // find its flags raised.  (Flags as some earlier launch left them, 0 once cleared.)
  long early = 0, cleared = 0, launches = 0;
  for (unsigned stages : {7u, 162u, 1922u}) {
    unsigned epoch = kSmallEpochLimit - 4 * stages, flag = epoch;
    for (unsigned long long gone = 0; gone < (2ull << 32); gone += stages, ++launches) {
      if (small_epoch_spent(epoch, stages)) {
        epoch = 0;
        flag = 0;
        ++cleared;
      }
      early += small_flag_reached(flag, epoch + 1) + small_flag_reached(flag, epoch + stages);
      early += !small_flag_reached(epoch + stages, epoch + stages);  // (and a raised one counts)
      epoch += stages;
    }
  }
  printf("%ld %ld %d\n", early, cleared, launches > 1000000);
}
"""


def test_flags_of_idle_launches_never_count_as_raised(tmp_path):
    early, cleared, enough = _run(tmp_path, EPOCHS)
    assert early == 0 and cleared >= 6 and enough


def test_flags_never_cleared_would_count_as_raised(tmp_path):
    """What the limit is for: without it the walk above finds stages that wait for nobody."""
    source = EPOCHS.replace("if (small_epoch_spent(epoch, stages))", "if (false)")
    assert source != EPOCHS and _run(tmp_path, source)[0] > 0
