// The compaction of a decode's active series by one workgroup: of the kernel that does nothing else (misc.hip), and of a round's workgroup
// that commits last (series_f32.hip).
#pragma once
#include "tsd_internal.h"

namespace tsd {

// list: the active series, ascending.  Returned, by lane 0 of the workgroup of W wavefronts: how many there are, and the most patches one
// of them still needs.  load: reads a word of active or committed.
template <int W, typename Load>
__device__ __forceinline__ int2 compact_step(const int* active, const int* committed, int T, int B, int* list, Load load) {
  __shared__ int wave_cnt[W], most[W];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  int base = 0, rem = 0;
  for (int b0 = 0; b0 < B; b0 += W * 64) {
    const int b = min(b0 + tid, B - 1), on_b = load(active + b), done = load(committed + b);
    const bool on = b0 + tid < B && on_b != 0;
    if (on) rem = max(rem, T - done);
    const unsigned long long m = __ballot(on);
    if (lane == 0) wave_cnt[w] = __popcll(m);
    __syncthreads();
    int off = base;
    for (int i = 0; i < W; ++i) {
      if (i < w) off += wave_cnt[i];
      base += wave_cnt[i];
    }
    if (on) list[off + __popcll(m & ((1ull << lane) - 1ull))] = b;
    __syncthreads();
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) rem = max(rem, __shfl_xor(rem, o));
  if (lane == 0) most[w] = rem;
  __syncthreads();
  if (tid == 0)
    for (int i = 1; i < W; ++i) rem = max(rem, most[i]);
  return make_int2(base, rem);
}

}  // namespace tsd
