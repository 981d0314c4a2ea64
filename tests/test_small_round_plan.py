"""Index rules of the resident decode kernel (csrc/small_round_plan.h), checked without a GPU: the header is plain C++, the program
below walks the reads of every product the kernel accepts."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_18191_amd", "csrc")

READS = r"""
#include <cstdio>
#include "small_round_plan.h"
using namespace tsd;

// How far behind the end of a row the reads of a product go: wavefront, part of its four slabs, k-step, 16-byte piece of a k-step.
long behind(const SmallPlan& d) {
  long most = 0;
  for (int wave = 0; wave < kSmallRoundWorkers && kSmallRoundWorkers * wave < d.used; ++wave)
    for (int part = 0; part < 4; ++part)
      for (int j = 0; j < d.per; ++j)
        for (int piece = 0; piece < 4; ++piece) {
          const long end = 2L * (slab_start(kSmallRoundWorkers * wave + part, d.per) + j * 32 + piece * 8 + 8 - d.K);
          if (end > most) most = end;
        }
  return most;
}

int main() {
  long products = 0, ragged = 0, bad = 0, overlaps = 0, most = 0;
  for (int K = 32; K <= 4096; K += 32)
    for (int N = 4; N <= 4096; N += 4)
      if (small_product_ok(K, N)) {
        const SmallPlan d = small_plan(K, N);
        const long b = behind(d);
        ++products;
        ragged += b > 0;
        bad += b > kSmallTail;
        if (b > most) most = b;
      }
  // the parts of a layer, 32 rows and a tail each, follow one another; no cache line of 128 bytes belongs to two
  for (int D = 64; D <= 1024; D += 64)
    for (int F = 32; F <= 4096; F += 32) {
      const size_t width[5] = {(size_t)D, (size_t)D, (size_t)D, (size_t)D, (size_t)F};
      const int part[5] = {kIn, kQuery, kMixed, kMid, kHidden};
      for (int i = 0; i < 5; ++i) {
        const size_t end = small_part_offset(D, part[i]) + kSmallRoundRows * width[i] * 2 + TAIL;
        overlaps += end > (i < 4 ? small_part_offset(D, part[i + 1]) : small_slab_bytes(D, F));
        overlaps += small_part_offset(D, part[i]) % 128 != 0;
      }
      overlaps += small_slab_bytes(D, F) % 128 != 0 || small_pass_bytes(3, D, F) % 128 != 0;
    }
  printf("%ld %ld %ld %ld %ld\n", products, ragged, bad, overlaps, most);
}
"""


def _run(tmp_path, source):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(source)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return [int(x) for x in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()]


def test_reads_stay_inside_their_part(tmp_path):
    products, ragged, bad, overlaps, most = _run(tmp_path, READS.replace("TAIL", "kSmallTail"))
    assert products > 10000 and ragged > 1000      # products whose last worker has fewer than four slabs are among them
    assert (bad, overlaps) == (0, 0) and most > 512


def test_parts_without_a_tail_would_be_read_early(tmp_path):
    """What the tail is for: laid out back to back, the parts are read from behind the one before."""
    back_to_back = READS.replace("bad += b > kSmallTail", "bad += b > 0").replace("TAIL", "0")
    assert _run(tmp_path, back_to_back)[2] > 0


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
