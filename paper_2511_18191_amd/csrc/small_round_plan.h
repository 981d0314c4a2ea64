// How the resident decode kernel (small_round.hip) deals its products out: sizes and index rules, in plain C++ so that they can be
// checked without a GPU (tests/test_small_round_plan.py).
#pragma once
#include <cstddef>

namespace tsd {

constexpr int kSmallRoundWorkgroups = 256;  // one per compute unit
constexpr int kSmallRoundRows = 32;         // rows of a pass at most
constexpr int kSmallRoundWorkers = 4;       // wavefronts that split a product's k range, four slabs each

struct SmallPlan {
  int K, units;   // units: workgroups that own columns of the product,
  int cs;         // 2^cs columns each (4, 8 or 16)
  int per, used;  // k-steps of 32 per slab, slabs
};

// Fewest columns per workgroup with which N columns fit the grid (0: they do not).
constexpr int columns_per_wg(int N) {
  for (int cw = 4; cw <= 16; cw *= 2)
    if (N % cw == 0 && N / cw <= kSmallRoundWorkgroups) return cw;
  return 0;
}

// The k range of a product is summed in slabs of consecutive k-steps of 32, each from zero, the slabs added in order: the
// order of the skinny kernel (gemm_skinny.hip: 16 wavefronts from K = 512 on, else 4), so that either gives the same bits.
constexpr SmallPlan small_plan(int K, int N) {
  const int nks = (K + 31) / 32, n = K >= 512 ? 16 : 4, cw = columns_per_wg(N);
  const int per = (nks + n - 1) / n;
  return SmallPlan{K, cw ? N / cw : 0, cw == 16 ? 4 : cw == 8 ? 3 : cw == 4 ? 2 : 0, per, (nks + per - 1) / per};
}

// A product of bf16 activations fits: its columns the grid, a worker's share of its weights eight pieces, its k range whole slabs.
constexpr bool small_product_ok(int K, int N) {
  const SmallPlan d = small_plan(K, N);
  return d.units && K % 32 == 0 && d.per * ((1 << d.cs) / 4) <= 8 && d.per * d.used * 32 == K;
}

// Worker `wave` reads slabs kSmallRoundWorkers * wave and the three behind it, four k ranges whose sums it keeps side by side.  A last
// worker with fewer than four reads past the end of its rows all the same (choosing the address takes 0.75 % of the kernel) and drops
// the sums.  That far behind row 31, and behind the last row of weights, nothing may lie that is written during the launch: a line
// that is read before it is published would be seen stale by the stage that needs it (see small_round.hip).
constexpr int slab_start(int slab, int per) { return slab * per * 32; }  // its first element in a row (and, of a count of slabs, their length)
// At most three slabs of eight k-steps, in whole 8 KB: the length decides on which memory channels the parts of a layer start (a round of
// one series through 24 layers of 1024 / of five through 8 of 512, us: back to back 687 / 315.0, tails of 2 KB 689 / 315.5, 4 KB
// 681 / 314.0, 8 KB 674 / 314.0, 16 KB 683 / 314.2).
constexpr int kSmallTail = 8192;
static_assert(3 * 8 * 64 <= kSmallTail, "");

// The exchange buffer: of a layer, the rows entering it, its queries, attention output, the rows between its two halves, hidden
// rows, each with a tail that nobody writes; of a pass, its layers and the fp32 residual.
enum SmallPart { kIn, kQuery, kMixed, kMid, kHidden };
constexpr size_t small_part_offset(int D, int part) { return (size_t)part * (kSmallRoundRows * 2 * D + kSmallTail); }
constexpr size_t small_slab_bytes(int D, int F) { return (size_t)kSmallRoundRows * (4 * D + F) * 2 + 5 * kSmallTail; }
constexpr size_t small_pass_bytes(int L, int D, int F) { return L * small_slab_bytes(D, F) + (size_t)kSmallRoundRows * D * 4; }

// The workgroups' flags count stages on from launch to launch: those of a launch run from `epoch` + 1, and a wait for `value` is over
// where flag - value is not negative as a signed number.  A launch that finds no series active advances the epoch and raises no
// flag, so a flag may lag by any number of launches; at 2^31 it would count as raised.  Before an epoch passes the limit the flags
// are cleared and it starts from 0 again.
constexpr unsigned kSmallEpochLimit = 1u << 30;
constexpr bool small_epoch_spent(unsigned epoch, unsigned stages) { return epoch > kSmallEpochLimit - stages; }
constexpr bool small_flag_reached(unsigned flag, unsigned value) { return (int)(flag - value) >= 0; }

}  // namespace tsd
