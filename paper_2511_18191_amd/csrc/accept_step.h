// The acceptance / correction / commit step of a round on a workgroup of 256 lanes per series: the body of accept_kernel (misc.hip),
// and of the kernel that follows the resident decode kernel (small_round.hip).
#pragma once
#include "philox.h"
#include "tsd_internal.h"

namespace tsd {

// One workgroup of four wavefronts per series.  Wavefront w forms the energies of positions w, w + 4, .. (reduced across
// lanes), then every wavefront for itself lets lane i own proposal i + 1: statistic, uniform, test; a ballot over the reject
// flags gives the first rejection.  The workgroup then writes the committed patches, the new pending / previous
// tokens and the cache lengths (rollback is metadata only: speculative KV entries past the accepted length are simply
// overwritten by the next round).
// The kernel is a chain of memory round trips, so there are three of them: the state words together with all patches (those
// of positions that turn out not to count included), then the rows to copy, then the stores.  One wavefront per series,
// positions in fours and the state words one after the other, took 10.6 us at 1024 series of 6 x 96, 7.9 at one of 4 x 96.
// Returned, by lane 0 alone: whether the series goes on, and how many patches it has committed.
__device__ __forceinline__ int2 accept_step(const AcceptP& p) {
  __shared__ float energy[2][16];
  if (p.n_dev && (int)blockIdx.x >= *p.n_dev) return make_int2(0, 0);
  const int b = p.act ? p.act[blockIdx.x] : (int)blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int K = p.K, P = p.P;
  const int KE = K > 0 ? K : 1;
  const bool stateful = p.len != nullptr;  // (a call without a handle: nothing committed before, no state kept)
  const int active = stateful ? p.active[b] : 1, r = p.round ? p.round[b] : 0, c0 = stateful ? p.committed[b] : 0;
  const float* X = p.X + (long)b * K * P;
  const float* MQ = p.mu_q + (long)b * K * P;
  const float* MP = p.mu_p + (long)b * (K + 1) * P;
  for (int i = wave; i < K; i += 8) {  // this wavefront's positions, two at a time
    const int i1 = min(i + 4, K - 1);
    float ep[2] = {0.f, 0.f}, eq[2] = {0.f, 0.f};
#pragma unroll 2
    for (int e = lane; e < P; e += 64) {
      const float x[2] = {X[i * P + e], X[i1 * P + e]}, mp[2] = {MP[i * P + e], MP[i1 * P + e]}, mq[2] = {MQ[i * P + e], MQ[i1 * P + e]};
      float wp = 1.f, wq = 1.f;
      if (p.inv2sp2_vec) {  // Mahalanobis energies of the diagonal surrogate, already halved
        wp = p.inv2sp2_vec[e];
        wq = p.inv2sq2_vec[e];
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const float dp = x[j] - mp[j], dq = x[j] - mq[j];
        if (p.inv2sp2_vec) {
          ep[j] = fmaf(dp * dp, wp, ep[j]);
          eq[j] = fmaf(dq * dq, wq, eq[j]);
        } else {
          ep[j] = fmaf(dp, dp, ep[j]);
          eq[j] = fmaf(dq, dq, eq[j]);
        }
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        ep[j] += __shfl_xor(ep[j], o);
        eq[j] += __shfl_xor(eq[j], o);
      }
    }
    if (lane == 0) {
      energy[0][i] = ep[0];
      energy[1][i] = eq[0];
      if (i + 4 < K) {
        energy[0][i + 4] = ep[1];
        energy[1][i + 4] = eq[1];
      }
    }
  }
  if (!active) {
    if (tid == 0) p.n_acc[b] = -1;
    if (tid < K) {
      p.ell[(long)b * KE + tid] = NAN;
      p.logu[(long)b * KE + tid] = NAN;
    }
    return make_int2(0, c0);
  }
  // a series with fewer than K patches left proposes and tests only as many positions as it
  // still needs: later ones could never be committed
  const int Kb = min(K, p.T - c0);
  __syncthreads();
  bool reject = false;
  float ell = NAN, logu = NAN, thr = 0.f;
  if (lane < Kb) {
    const float my_ep = energy[0][lane], my_eq = energy[1][lane];
    // Eq. 5 with per-dimension energies ||.||^2 / P
    if (p.threshold) {
      // threshold rule: ||x - mu_p||_d^2 <= sigma_p^2, written as ell >= -1/2 so that the recorded
      // pair (ell, log u) shows how close to the boundary the decision was
      ell = p.temper * (p.inv2sp2_vec ? -(my_ep / (float)P) : -(my_ep / (float)P) * p.inv2sp2);
      logu = -0.5f;
    } else {
      if (p.inv2sp2_vec)
        ell = p.temper * (-(my_ep / (float)P) + (my_eq / (float)P) + p.logdet_dev[0]);
      else
        ell = p.temper * (-(my_ep / (float)P) * p.inv2sp2 + (my_eq / (float)P) * p.inv2sq2 + p.logdet);
      unsigned w = philox_word0((unsigned)b, (unsigned)r, (unsigned)(lane + 1), 0u, p.key0, p.key1);
      float u = word_uniform(w);
      logu = logf(u);
    }
    thr = (p.log_alpha_override <= 0.f) ? p.log_alpha_override : fminf(0.f, ell);
    reject = !(logu <= thr);
  }
  const unsigned long long rej = __ballot(reject);
  const int n_free = rej ? (int)__builtin_ctzll(rej) : Kb;  // leading accepts
  const int tested = n_free + (n_free < Kb ? 1 : 0);
  const bool is_tested = lane < tested;
  const unsigned long long near = __ballot(is_tested && fabsf(thr - logu) < 1e-4f);
  int n = n_free;
  if (p.forced) {
    int f = p.forced[b];
    if (f >= 0 && f <= Kb) n = f;
  }
  if (p.mode == 1) {  // synchronised round, first launch: only the minimum over the series
    if (tid == 0) atomicMin(p.sync, n);
    return make_int2(1, c0);
  }
  if (p.mode == 2) n = min(n, *p.sync);
  if (tid < K && p.ell) p.ell[(long)b * KE + tid] = is_tested ? ell : NAN;
  if (tid < K && p.logu) p.logu[(long)b * KE + tid] = is_tested ? logu : NAN;
  const int L = n + 1;
  const int Lc = min(L, p.T - c0);
  float* fc = p.forecast + ((long)b * p.T + c0) * P;
  for (int j = wave; j < min(Lc, n); j += 4)
    for (int e = lane; e < P; e += 64) fc[j * P + e] = X[j * P + e];
  if (p.clear_rest)
    for (int e = Lc * P + tid; e < (p.T - c0) * P; e += 256) fc[e] = 0.f;
  // corrected (n < K) or bonus (n = K) patch: the target mean, plus r * eps when fallback noise is on
  for (int e = tid; e < P; e += 256) {
    float t = MP[n * P + e];
    const float last = stateful ? (n >= 1 ? X[(n - 1) * P + e] : p.pending[(long)b * P + e]) : 0.f;
    if (p.fallback_r > 0.f)
      t += p.fallback_r * normal_draw((unsigned)b, (unsigned)r, (unsigned)(n + 1), kStreamFallback, e, p.key0, p.key1);
    if (n < Lc) fc[n * P + e] = t;
    if (stateful) {
      p.prev[(long)b * P + e] = last;
      p.pending[(long)b * P + e] = t;
    }
  }
  if (tid == 0) {
    p.n_acc[b] = n_free;
    if (stateful) {
      p.len[b] += Lc;
      p.committed[b] = c0 + Lc;
      p.round[b] = r + 1;
      p.active[b] = (c0 + Lc < p.T) ? 1 : 0;
      long long* st = p.stat + (long)b * 5;
      st[0] += 1;
      st[1] += tested;
      st[2] += n_free;
      st[3] += Lc;
      st[4] += __popcll(near);
    }
  }
  return make_int2(c0 + Lc < p.T ? 1 : 0, c0 + Lc);
}

}  // namespace tsd
