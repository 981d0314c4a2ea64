// Passes of small fp32 models, a series per workgroup: all draft steps of a round, the verification pass, the acceptance step and
// the compaction behind it as one launch, and the context pass of both models as another.
//
// Kernel by kernel such a round is some 35 dependent launches of 4 to 6 us that each touch a few KB.  Series never exchange
// anything inside a round, so a workgroup of 8 wavefronts takes its series through every stage with barriers of its own in
// place of launches; residual, activations, patches and the layer's keys and values sit in LDS.  8 series through 2 layers of 64 (draft 1 of
// 32, 32 patches of context, K = 4): 544 us a forecast kernel by kernel, 165 to 177 here; a round of four proposals 64 us, of one 39, the
// context 34.  What bounds it: the chain of latencies of a stage (a barrier, LDS, 8 to 64 matrix instructions of 32 clocks, an epilogue:
// 1 to 2 us), not bytes.  Of a round's wavefront cycles 58 % wait (barriers, LDS, loads), 16 % for an instruction to issue; the matrix cores
// in use are busy for 14 % of the time, bank conflicts take 4 % of a compute unit's clocks, and the weights come from behind the L2s, each
// of which has them to fetch anew in a launch (22 % L2 hits, 390 clocks a read).
//
//   * Sizes are template parameters (Shape): known only at run time they made a product's stage some 1000 instructions long, 4000
//     clocks for 500 of matrix instructions, and a round of 127 us.
//   * A wavefront takes every 8th block of 16 columns of a product and its whole k range: v_mfma_f32_16x16x4_f32, k in ascending
//     order as in gemm_f32.hip, same bits.  The weights are a second copy in the order the lanes want them (16 bytes of a row's
//     16-wide k-run per lane and load, a KB per load); activations in LDS have the four k of a run that belong to a lane next to
//     each other (run_pos).
//   * The first loads of a wavefront's next product are issued as soon as its registers are free, before the epilogue and the
//     barrier in between (a bare barrier: weight loads stay in flight across it).
//   * QKV columns are packed in rotary-pair order: a block is eight columns of the first half of a head and their partners.
//   * Attention: up to eight queries a wavefront per (query, head), the sums of attn_kernel (attn.hip) in the same order; more of them
//     16 at a time on the matrix cores (attend16), with the same bits.
#include <algorithm>
#include <type_traits>

#include "accept_step.h"
#include "compact_step.h"
#include "series_plan.h"
#include "tsd_internal.h"

namespace tsd {

namespace {

constexpr int kWaves = 8, kThreads = kWaves * 64;
constexpr int kChunk = 8;   // 16-wide k-runs whose weights are in registers at a time

// Position of column c of an activation row in LDS: within a run of 16, lane group c % 4's four columns next to each other.
__host__ __device__ constexpr int run_pos(int c) { return (c & ~15) | ((c & 3) << 2) | ((c >> 2) & 3); }
__host__ __device__ constexpr int up16(int n) { return (n + 15) & ~15; }

// LDS of a workgroup, in words.  `rows`: of a pass, a multiple of 16; `tokens`: a launch has patches and rotary factors for at a
// time, for as many models; S: cached tokens at most.
struct Carve {
  int x, cos, sin, patch, odd, table, probs, shared, total;
};
// A wavefront's attention weights: of one query, or of 16 and 32 keys.
constexpr int kTileKeys = 64, kLdProbs = 36;
__host__ __device__ constexpr int probs_words(int S) { return up16(S) > 16 * kLdProbs ? up16(S) : 16 * kLdProbs; }
// Words of the part that one stage after the other uses: queries, attention output, keys and values; hidden rows.
__host__ __device__ constexpr int shared_words(int D, int F, int rows, int S) {
  const int attn = (2 * rows + 2 * S) * (D + 4), hid = rows * (F + 4);
  return attn > hid ? attn : hid;
}
__host__ __device__ constexpr Carve carve_of(int D, int half, int P, int rows, int tokens, int models, int S, int shared) {
  Carve c{};
  c.x = 0;
  c.cos = rows * (D + 4);
  c.sin = c.cos + models * tokens * half;
  c.patch = c.sin + models * tokens * half;
  c.odd = c.patch + tokens * (up16(P) + 4);
  c.table = c.odd + 4;
  c.probs = c.table + 64;
  c.shared = c.probs + kWaves * probs_words(S);
  c.total = c.shared + shared;  // (a pass of fewer than its rows reads on behind its rotary factors: they are in front)
  return c;
}

__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The weights of a product: blocks of 16 columns, each its 16-wide k-runs of 1 KB one after the other.  A wavefront takes every 8th
// block; Frags holds up to kChunk runs of one.
struct Frags {
  float4 w[kChunk];
};
template <int N>
__device__ __forceinline__ void load_runs(const float* W, int first, int lane, Frags& f) {  // `first`: run number in the product
  const float4* src = reinterpret_cast<const float4*>(W) + first * 64 + lane;
#pragma unroll
  for (int t = 0; t < N; ++t) f.w[t] = src[t * 64];
}
__device__ __forceinline__ void load_some_runs(const float* W, int first, int n, int lane, Frags& f) {
  const float4* src = reinterpret_cast<const float4*>(W) + first * 64 + lane;
#pragma unroll
  for (int t = 0; t < kChunk; ++t)
    if (t < n) f.w[t] = src[t * 64];
}

// acc += N runs of the rows of A (whose reads go out together) times f.
template <int RT, int N>
__device__ __forceinline__ void add_runs(const float* a0, int ld, const float4* w, f32x4* acc) {
  float4 a[N][RT];
#pragma unroll
  for (int t = 0; t < N; ++t)
#pragma unroll
    for (int i = 0; i < RT; ++i) a[t][i] = *reinterpret_cast<const float4*>(a0 + i * 16 * ld + t * 16);
#pragma unroll
  for (int t = 0; t < N; ++t) {
#pragma unroll
    for (int i = 0; i < RT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t][i].x, w[t].x, acc[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < RT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t][i].y, w[t].y, acc[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < RT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t][i].z, w[t].z, acc[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < RT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t][i].w, w[t].w, acc[i], 0, 0, 0);
  }
}

template <int RT>
__device__ __forceinline__ void clear(f32x4* acc) {
#pragma unroll
  for (int i = 0; i < RT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// Rows of A (LDS, LD words apart) times the wavefront's blocks: f[0] holds the first loads; later ones go to f[1] and f[0] in turn, and
// next() brings those of the next product to f[0].
// fin(block, acc): lane l holds rows 16 i + 4 (l / 16) + r, column l % 16 of the block in acc[i][r].
template <int RT, int BLOCKS, int RUNS, int LD, typename Next, typename Fin>
__device__ __forceinline__ void product(const float* W, const float* A, int wave, int lane, Frags* f, Next next, Fin fin) {
  constexpr int NB = (BLOCKS + kWaves - 1) / kWaves, N = RUNS < kChunk ? RUNS : kChunk, NC = RUNS / N;
  static_assert(RUNS % N == 0, "whole chunks");
  if (wave >= BLOCKS) {
    next();
    return;
  }
  const float* a0 = A + (lane & 15) * LD + (lane >> 4) * 4;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int blk = wave + b * kWaves;
    if (BLOCKS % kWaves && b + 1 == NB && b > 0 && blk >= BLOCKS) break;
    f32x4 acc[RT];
    clear<RT>(acc);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int i = b * NC + c;  // chunk number
      if (c + 1 < NC) load_runs<N>(W, blk * RUNS + (c + 1) * N, lane, f[(i + 1) & 1]);
      else if (b + 1 < NB && blk + kWaves < BLOCKS) load_runs<N>(W, (blk + kWaves) * RUNS, lane, f[(i + 1) & 1]);
      add_runs<RT, N>(a0 + c * N * 16, LD, f[i & 1].w, acc);
    }
    if (b + 1 == NB || blk + kWaves >= BLOCKS) next();
    fin(blk, acc);
  }
}

// Sums over l ^ 32, l ^ 16, .. in that order, lanes exchanged in registers: within 16 lanes a rotation reaches the lane wanted or one
// that holds the same sum already.  (By shuffles through LDS a step took 100 cycles; there are 12 in a row per query.)
template <typename N>
__device__ __forceinline__ float rotate16(float v, N) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N::value, 0xf, 0xf, false));
}
template <typename Op>
__device__ __forceinline__ float over_halves(float v, Op op) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(p[0]), __uint_as_float(p[1]));
}
template <typename Op>
__device__ __forceinline__ float over_rows(float v, Op op) {  // l ^ 16
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(p[0]), __uint_as_float(p[1]));
}
template <typename Op>
__device__ __forceinline__ float over16(float v, Op op) {
  v = op(v, rotate16(v, std::integral_constant<int, 8>{}));
  v = op(v, rotate16(v, std::integral_constant<int, 4>{}));
  v = op(v, rotate16(v, std::integral_constant<int, 2>{}));
  return op(v, rotate16(v, std::integral_constant<int, 1>{}));
}
template <typename Op>
__device__ __forceinline__ float over_wave(float v, Op op) {
  return over16(over_rows(over_halves(v, op), op), op);
}
struct Add {
  __device__ __forceinline__ float operator()(float a, float b) const { return a + b; }
};
struct Max {
  __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};

// RMSNorm scales of the rows of x: lane l gets that of row 16 i + l % 16 in rs[i].  Per row four partial sums, one per 16-byte
// piece of a run, combined as (P0 + P2) + (P1 + P3): the order of gemm_f32.hip.
template <int RT, int D>
__device__ __forceinline__ void row_scales(const float* x, int lane, float* rs) {
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    const float* row = x + (16 * i + (lane & 15)) * (D + 4) + (lane >> 4);
    float ss = 0.f;
#pragma unroll
    for (int t = 0; t < D; t += 16) {
      const float f0 = row[t], f1 = row[t + 4], f2 = row[t + 8], f3 = row[t + 12];
      ss += f0 * f0 + f1 * f1 + f2 * f2 + f3 * f3;
    }
    const float s = over_rows(over_halves(ss, Add{}), Add{});
    rs[i] = rsqrtf(s / (float)D + kRmsEps);
  }
}
// ... applied to a block's sums
template <int RT>
__device__ __forceinline__ void scale_rows(const float* rs, int lane, f32x4* acc) {
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[i][r] *= __shfl(rs[i], 4 * (lane >> 4) + r);
}

// One query of one head over keys 0 .. nkeys - 1 by a wavefront: q and out are the head's columns, K and V those of token 0.
template <int HD>
__device__ __forceinline__ void attend(const float* q, const float* Ks, const float* Vs, int ld, int nkeys, float* ps, float* out_row, int c0, int lane) {
  constexpr int G = 64 / HD;
  const int nk4 = (nkeys + 3) & ~3;
  float m = -INFINITY;
  for (int s = lane; s < nk4; s += 64) {
    float sc = 0.f;
    const float* kr = Ks + min(s, nkeys - 1) * ld;
#pragma unroll
    for (int e = 0; e < HD; e += 4) {
      const float4 k = *reinterpret_cast<const float4*>(kr + e), qq = *reinterpret_cast<const float4*>(q + e);
      sc = fmaf(k.x, qq.x, sc);
      sc = fmaf(k.y, qq.y, sc);
      sc = fmaf(k.z, qq.z, sc);
      sc = fmaf(k.w, qq.w, sc);
    }
    sc = s < nkeys ? sc : -INFINITY;
    ps[s] = sc;
    m = fmaxf(m, sc);
  }
  m = over_wave(m, Max{});
  float sum = 0.f;
  for (int s = lane; s < nk4; s += 64) {  // (a lane's own scores)
    const float e = __expf(ps[s] - m);
    ps[s] = e;
    sum += e;
  }
  const float inv = 1.f / over_wave(sum, Add{});
  wave_lds_order();
  const int d = lane % HD, sg = lane / HD;
  float acc = 0.f;
  for (int s4 = sg * 4; s4 < nk4; s4 += 4 * G) {
    const float4 pp = *reinterpret_cast<const float4*>(ps + s4);
    float vv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) vv[u] = s4 + u < nkeys ? Vs[(s4 + u) * ld + d] : 0.f;
    acc = fmaf(pp.x, vv[0], acc);
    acc = fmaf(pp.y, vv[1], acc);
    acc = fmaf(pp.z, vv[2], acc);
    acc = fmaf(pp.w, vv[3], acc);
  }
  if constexpr (HD == 16) acc = over_rows(acc, Add{});
  if constexpr (HD <= 32) acc = over_halves(acc, Add{});
  if (sg == 0) out_row[run_pos(c0 + d)] = acc * inv;
  wave_lds_order();
}

// The same for the 16 queries q, q + ld, .. of a head (`rows` of them there are) on the matrix cores, key `base` the first query's own,
// S keys in all, at most kTileKeys: the same bits.  Scores: a matrix instruction adds its four products in ascending order, as the
// chain above does.  Sums of the exponentials: a lane holds key l % 16 of a block of 16, and the four blocks of 64 keys are what
// the lanes 16 apart held.  Output: four keys per instruction, the 64 / HD groups of keys in sums of their own, added in their order.
// A weight of a key the query does not see is zero, and its value has to be finite (see run_series_pass).
// ps: 16 x kLdProbs words of this wavefront's.
template <int HD, int LDX>
__device__ __forceinline__ void attend16(const float* q, const float* Ks, const float* Vs, int base, int S, float* ps, float* out, int c0, int lane) {
  constexpr int NKB = kTileKeys / 16, G = 64 / HD, CB = HD / 16;
  const int l15 = lane & 15, lq = lane >> 4, n_kb = (S + 15) >> 4;
  f32x4 sc[NKB];
  {
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) sc[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
    float qf[HD / 4];
#pragma unroll
    for (int e = 0; e < HD / 4; ++e) qf[e] = q[l15 * LDX + 4 * e + lq];
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
      if (kb >= n_kb) break;
      const float* kr = Ks + min(16 * kb + l15, S - 1) * LDX + lq;
#pragma unroll
      for (int e = 0; e < HD / 4; ++e) sc[kb] = __builtin_amdgcn_mfma_f32_16x16x4f32(qf[e], kr[4 * e], sc[kb], 0, 0, 0);
    }
  }
  // this lane: queries 4 lq + r, keys 16 kb + l15
  float inv[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int seen = min(base + 4 * lq + r, S - 1);
    float m = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
      if (kb >= n_kb) break;
      if (16 * kb + l15 > seen) sc[kb][r] = -INFINITY;
      m = fmaxf(m, sc[kb][r]);
    }
    m = over16(m, Max{});
    float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
      if (kb >= n_kb) break;
      sc[kb][r] = __expf(sc[kb][r] - m);
      part[kb & 3] += sc[kb][r];
    }
    inv[r] = 1.f / over16((part[0] + part[2]) + (part[1] + part[3]), Add{});
  }
  f32x4 o[4];  // group g, block of 16 output columns cb: o[g * CB + cb]
  clear<4>(o);
#pragma unroll
  for (int k2 = 0; k2 < NKB / 2; ++k2) {  // 32 keys at a time through LDS
    if (2 * k2 >= n_kb) break;
    wave_lds_order();
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) ps[(4 * lq + r) * kLdProbs + 16 * j + l15] = 2 * k2 + j < n_kb ? sc[2 * k2 + j][r] : 0.f;
    wave_lds_order();
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int key = 32 * k2 + 4 * j + lq;
      const float w = ps[l15 * kLdProbs + 4 * j + lq];
      const float* vr = Vs + min(key, S - 1) * LDX + l15;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        const float v = key < S ? vr[16 * cb] : 0.f;
        o[j % G * CB + cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, v, o[j % G * CB + cb], 0, 0, 0);
      }
    }
  }
  wave_lds_order();
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    if constexpr (G == 4) o[cb] = (o[0] + o[1]) + (o[2] + o[3]);
    if constexpr (G == 2) o[cb] = o[cb] + o[CB + cb];
#pragma unroll
    for (int r = 0; r < 4; ++r) out[(4 * lq + r) * LDX + run_pos(c0 + 16 * cb + l15)] = o[cb][r] * inv[r];
  }
}

// One pass of one series: nq tokens (at most 16 RT) at positions base, base + 1, .., which are tokens first, first + 1, .. of the launch
struct SeriesPass {
  int nq, base, first;
  float* out;  // head outputs of tokens t_skip, .. (NULL: no head)
  int t_skip;
  int keep;    // they are the patches of tokens keep, .. of the launch (0: they are not)
};

// The model sizes there are kernels for: widths of 32, 64 and 128 with a four times as wide FFN.
template <int D_, int HD_>
struct Shape {
  static constexpr int D = D_, F = 4 * D_, HD = HD_, H = D_ / HD_, HALF = HD_ / 2, DB = D_ / 16, FB = F / 16, LDX = D_ + 4, LDH = F + 4;
};

__device__ __forceinline__ void prefetch_embed(const SeriesModel& m, int P, int wave, int lane, Frags* f) {
  const int runs = up16(P) >> 4;
  if (wave < m.D >> 4) load_some_runs(m.We, wave * runs, runs, lane, f[0]);
}

// f[0] holds the first loads of the model's embedding; after() brings those of the next pass's.
template <typename M, int RT, typename After>
__device__ __forceinline__ void run_series_pass(const SeriesP& p, const SeriesModel& m, const SeriesPass& ps, float* lds, Frags* f, After after) {
  constexpr int D = M::D, LDX = M::LDX, LDH = M::LDH, HD = M::HD, H = M::H, HALF = M::HALF, DB = M::DB, FB = M::FB, R = 16 * RT;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // (an opaque copy: keeps the address arithmetic of all shapes from being hoisted out of the passes)
  int lane = tid & 63, l15 = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int P = p.P, nq = ps.nq, base = ps.base, S = base + nq, ldp = up16(P) + 4, pr = up16(P) >> 4;
  const Carve c = carve_of(p.D_max, p.half_max, P, R, p.tokens, p.models, p.S_max, 0);
  const int rope = (p.models == 2 ? m.draft * p.tokens * p.half_max : 0) + ps.first * HALF;
  float *x = lds + c.x, *cs = lds + c.cos + rope, *sn = lds + c.sin + rope, *shared = lds + c.shared, *patch = lds + c.patch;
  const int* table = reinterpret_cast<const int*>(lds + c.table);
  float *q = shared, *att = q + R * LDX, *Ks = att + R * LDX, *Vs = Ks + S * LDX, *hid = shared;
  float* probs = lds + c.probs + wave * probs_words(p.S_max);
  volatile int* odd = reinterpret_cast<int*>(lds + c.odd);  // a value of the pass's tokens is not finite
  const int plane = p.PT * HD;  // a head's keys of a page; its values are H planes on
  auto token_at = [&](int tok) { return kv_token(table[tok >> p.pt_shift], tok & (p.PT - 1), H, p.PT, HD); };
  // keys and values of earlier passes, 16 bytes at a time: half a wavefront the keys, half the values of FIT tokens, the wavefronts
  // tokens in turn
  constexpr int C4 = D / 4, FIT = 32 / C4, U = 4, STEP = kWaves * FIT;
  const int cc = (lane & 31) % C4, tok_first = wave * FIT + (lane & 31) / C4;
  const int old_from = ((lane >> 5) * H + cc / (HD / 4)) * plane + cc % (HD / 4) * 4;
  float* old_to = (lane < 32 ? Ks : Vs) + cc * 4;
  auto fetch = [&](const float* pool, int tok0, float4* old) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      old[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (tok0 + u * STEP < base) old[u] = *reinterpret_cast<const float4*>(pool + (old_from + token_at(tok0 + u * STEP)));
    }
  };
  auto put = [&](int tok0, const float4* old) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (tok0 + u * STEP < base) *reinterpret_cast<float4*>(old_to + (tok0 + u * STEP) * LDX) = old[u];
  };
  auto x_at = [&](int blk) { return x + 4 * lq * LDX + 16 * blk + run_pos(l15); };
  auto add_to_x = [&](int blk, f32x4* acc) {
    float* to = x_at(blk);
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][r] = to[(16 * i + r) * LDX] + acc[i][r];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) to[(16 * i + r) * LDX] = acc[i][r];
  };
  const float* W = m.layers;
  auto first_of = [&](const float* Wn, int blocks, auto runs) {
    constexpr int RUNS = decltype(runs)::value;
    if (wave < blocks) load_runs < RUNS < kChunk ? RUNS : kChunk > (Wn, wave * RUNS, lane, f[0]);
  };
  using Db = std::integral_constant<int, DB>;
  using Fb = std::integral_constant<int, FB>;

  float4 old[U];
  fetch(m.kv_pool, tok_first, old);
  if (wave < DB) {
    const float* a0[RT];  // (rows past nq: the last one's patch)
#pragma unroll
    for (int i = 0; i < RT; ++i) a0[i] = patch + (ps.first + min(16 * i + l15, nq - 1)) * ldp + lq * 4;
    f32x4 acc[RT];
    clear<RT>(acc);
    for (int t0 = 0; t0 < pr; t0 += kChunk) {
      if (t0) load_some_runs(m.We, wave * pr + t0, pr - t0, lane, f[0]);
#pragma unroll
      for (int t = 0; t < kChunk; ++t)
        if (t0 + t < pr) {
#pragma unroll
          for (int i = 0; i < RT; ++i) add_runs<1, 1>(a0[i] + (t0 + t) * 16, 0, &f[0].w[t], acc + i);
        }
    }
    first_of(W, 3 * DB, Db{});
    float* to = x_at(wave);
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) to[(16 * i + r) * LDX] = acc[i][r];
  } else {
    first_of(W, 3 * DB, Db{});
  }
  lds_barrier();

#pragma unroll 1
  for (int l = 0; l < m.L; ++l, W += m.layer_words) {
    asm volatile("" : "+v"(lane));  // (nor out of the layers)
    l15 = lane & 15;
    lq = lane >> 4;
    float* pool = m.kv_pool + (size_t)l * m.layer_pool_elems;
    {
      float rs[RT];
      row_scales<RT, D>(x, lane, rs);
      product<RT, 3 * DB, DB, LDX>(W, x, wave, lane, f, [&] { first_of(W + m.o_out, DB, Db{}); }, [&](int blk, f32x4* acc) {
        scale_rows<RT>(rs, lane, acc);
        constexpr int BPH = HD / 16;
        const int hs = blk / BPH, i8 = blk % BPH * 8 + (l15 & 7), which = hs / H, h = hs % H;
        const int col = h * HD + i8 + (l15 < 8 ? 0 : HALF);
        if (which < 2) {
          const float sg = l15 < 8 ? -1.f : 1.f;
#pragma unroll
          for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float pv = rotate16(acc[i][r], std::integral_constant<int, 8>{});
              const int at = (16 * i + 4 * lq + r) * HALF + i8;  // (rows past nq: whatever is there, dropped)
              acc[i][r] = acc[i][r] * cs[at] + sg * pv * sn[at];
            }
        }
        if (which == 0) {
#pragma unroll
          for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) q[(16 * i + 4 * lq + r) * LDX + col] = acc[i][r] * m.scale;
        } else {
          float* to = (which == 1 ? Ks : Vs) + base * LDX + col;
          float* cache = pool + ((which - 1) * H + h) * plane + (col - h * HD);
#pragma unroll
          for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int row = 16 * i + 4 * lq + r;
              if (row < nq) {
                // (a value that is none: only queries that see its key may, and attention takes them one by one)
                if (which == 2 && !(fabsf(acc[i][r]) < INFINITY)) *odd = 1;
                to[row * LDX] = acc[i][r];
                cache[token_at(base + row)] = acc[i][r];
              }
            }
        }
      });
    }
    put(tok_first, old);
    for (int tok = tok_first + U * STEP; tok < base; tok += U * STEP) {
      fetch(pool, tok, old);
      put(tok, old);
    }
    lds_barrier();
    // ---- attention ----
    // (Up to eight queries a wavefront each is the faster way, more of them the matrix cores.  Against the other way, timed when the rule was
    // made: a round of 5 tokens 61 us / 70, a context of 31 33 us / 48.)
    if (nq > 8 && S <= kTileKeys && !*odd) {
      for (int t = wave; t < ((nq + 15) >> 4) * H; t += kWaves) {
        const int row = t / H * 16, c0 = t % H * HD;
        attend16<HD, LDX>(q + row * LDX + c0, Ks + c0, Vs + c0, base + row, S, probs, att + row * LDX, c0, lane);
      }
    } else {
      for (int t = wave; t < nq * H; t += kWaves) {
        const int row = t / H, c0 = t % H * HD;
        attend<HD>(q + row * LDX + c0, Ks + c0, Vs + c0, LDX, base + row + 1, probs, att + row * LDX, c0, lane);
      }
    }
    lds_barrier();
    product<RT, DB, DB, LDX>(W + m.o_out, att, wave, lane, f, [&] { first_of(W + m.o_up, FB, Db{}); }, add_to_x);
    lds_barrier();
    {
      float rs[RT];
      row_scales<RT, D>(x, lane, rs);
      product<RT, FB, DB, LDX>(W + m.o_up, x, wave, lane, f, [&] { first_of(W + m.o_down, DB, Fb{}); }, [&](int blk, f32x4* acc) {
        scale_rows<RT>(rs, lane, acc);
        float* to = hid + 4 * lq * LDH + 16 * blk + run_pos(l15);
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) to[(16 * i + r) * LDH] = gelu_tanh(acc[i][r]);
      });
    }
    if (l + 1 < m.L) fetch(pool + m.layer_pool_elems, tok_first, old);  // (put down behind the next QKV product)
    lds_barrier();
    product<RT, DB, FB, LDH>(W + m.o_down, hid, wave, lane, f, [&] {
      if (l + 1 < m.L) first_of(W + m.layer_words, 3 * DB, Db{});
      else if (ps.out) first_of(m.Wh, pr, Db{});
      else after();
    }, add_to_x);
    lds_barrier();
  }
  if (ps.out) {
    float rs[RT];
    row_scales<RT, D>(x, lane, rs);
    const float* a0 = x + l15 * LDX + lq * 4;
    if (wave >= pr) after();
    for (int blk = wave; blk < pr; blk += kWaves) {
      if (blk != wave) load_runs<DB>(m.Wh, blk * DB, lane, f[0]);
      f32x4 acc[RT];
      clear<RT>(acc);
      add_runs<RT, DB>(a0, LDX, f[0].w, acc);
      if (blk + kWaves >= pr) after();
      scale_rows<RT>(rs, lane, acc);
      const int col = 16 * blk + l15;
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * i + 4 * lq + r;
          if (col < P && row < nq && row >= ps.t_skip) {
            ps.out[(row - ps.t_skip) * P + col] = acc[i][r];
            if (ps.keep) patch[(ps.keep + row - ps.t_skip) * ldp + 16 * blk + run_pos(l15)] = acc[i][r];
          }
        }
    }
  }
  __syncthreads();  // the pass's cache rows and outputs are there for this workgroup
}

// The number of a model's Shape (-1: there is none).
constexpr int shape_of(int D, int H, int F) {
  if (F != 4 * D || H < 1 || D % H) return -1;
  const int hd = D / H, h = hd == 16 ? 0 : hd == 32 ? 1 : hd == 64 ? 2 : 3;
  return h > 2 || hd > D ? -1 : D == 32 ? h : D == 64 ? 2 + h : D == 128 ? 5 + h : -1;
}
template <int RT, typename After>
__device__ __forceinline__ void run_any_pass(const SeriesP& p, const SeriesModel& m, const SeriesPass& ps, float* lds, Frags* f, After after) {
  switch (m.shape) {
    case 0: return run_series_pass<Shape<32, 16>, RT>(p, m, ps, lds, f, after);
    case 1: return run_series_pass<Shape<32, 32>, RT>(p, m, ps, lds, f, after);
    case 2: return run_series_pass<Shape<64, 16>, RT>(p, m, ps, lds, f, after);
    case 3: return run_series_pass<Shape<64, 32>, RT>(p, m, ps, lds, f, after);
    case 4: return run_series_pass<Shape<64, 64>, RT>(p, m, ps, lds, f, after);
    case 5: return run_series_pass<Shape<128, 16>, RT>(p, m, ps, lds, f, after);
    case 6: return run_series_pass<Shape<128, 32>, RT>(p, m, ps, lds, f, after);
    case 7: return run_series_pass<Shape<128, 64>, RT>(p, m, ps, lds, f, after);
  }
}

// What the passes of a launch share: patches of its tokens, as far as they are there before it, their rotary factors, the page table.
// Token t sits at position pos + t; model: the first of p.models; patch_of(t): its patch (NULL: a pass of the launch makes it).
template <int RT, typename Patch>
__device__ __forceinline__ void set_up(const SeriesP& p, int model, int b, int pos, int n, float* lds, Patch patch_of) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const Carve c = carve_of(p.D_max, p.half_max, p.P, 16 * RT, p.tokens, p.models, p.S_max, 0);
  int* table = reinterpret_cast<int*>(lds + c.table);
  if (tid < p.pt_stride) table[tid] = p.page_table[(long)b * p.pt_stride + tid];
  if (tid == 64) reinterpret_cast<int*>(lds + c.odd)[0] = 0;
  const int n4 = up16(p.P) >> 2;
  for (int t = wave; t < n; t += kWaves) {
    const float* src = patch_of(t);
    for (int k4 = lane; k4 < n4; k4 += 64) {
      const bool in = k4 < p.P >> 2;
      if (!src && in) continue;
      const float4 v = in ? *reinterpret_cast<const float4*>(src + k4 * 4) : make_float4(0.f, 0.f, 0.f, 0.f);
      float* to = lds + c.patch + t * (n4 * 4 + 4) + (k4 & ~3) * 4 + (k4 & 3);
      to[0] = v.x;
      to[4] = v.y;
      to[8] = v.z;
      to[12] = v.w;
    }
  }
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    if (w == p.models) break;
    const SeriesModel& m = p.m[model + w];
    const int at = w * p.tokens * p.half_max;
    for (int i = tid; i < n * m.half; i += kThreads) {  // (positions are consecutive)
      lds[c.cos + at + i] = m.rope_cos[pos * m.half + i];
      lds[c.sin + at + i] = m.rope_sin[pos * m.half + i];
    }
  }
  __syncthreads();
}

// By the workgroup of a round that commits last.  What the others committed has gone through to memory before they were counted; it is
// read past the caches.
__device__ __forceinline__ void compact(const CompactP& c) {
  const int seq = c.count[4] + 1;
  const int2 now = compact_step<4>(c.active, c.committed, c.T, c.B, c.list,
                                   [](const int* a) { return __hip_atomic_load(const_cast<int*>(a), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); });
  if (threadIdx.x == 0) {
    c.count[0] = now.x;
    c.count[1] = now.y;
    c.count[4] = seq;
    // (the launch's number goes last: the caller watches it)
    __hip_atomic_store(&c.host[0], now.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&c.host[1], now.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __hip_atomic_store(&c.host[2], seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

}  // namespace

// Slot blockIdx.x of the list: the draft steps (p.phases & 1), the target pass (& 2), the acceptance step (& 4), and behind the
// last of them the compaction (c.host not NULL).
template <int RT>
__global__ __launch_bounds__(kThreads) void series_round_kernel(const SeriesP p, const AcceptP a, const CompactP c) {
  extern __shared__ __attribute__((aligned(16))) float series_lds[];
  const int n = p.counts ? min(p.counts[0], p.n) : p.n;
  if ((int)blockIdx.x >= n) {
    if (n == 0 && blockIdx.x == 0 && c.host && threadIdx.x < 256) compact(c);  // (nobody is left; the caller waits for the count)
    return;
  }
  const int b = p.act ? p.act[blockIdx.x] : (int)blockIdx.x;
  const int Kr = p.follow_need ? max(1, min(p.K, p.counts[1])) : p.K;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  Frags f[2];
  prefetch_embed(p.m[p.phases & 1 ? 1 : 0], p.P, wave, tid & 63, f);
  const int len = p.len[b], P = p.P;
  float* X = p.X + (long)b * p.x_stride;
  // tokens of the launch: the one before the pending one, the pending one, the proposals
  set_up<RT>(p, 0, b, len - 1, p.step_only ? 2 : Kr + 2, series_lds, [&](int t) -> const float* {
    if (t < 2) return (t ? p.pending : p.prev) + (long)b * P;
    return p.phases & 1 ? nullptr : X + (t - 2) * P;
  });
  const int steps = p.phases & 1 ? Kr : 0, passes = steps + (p.phases & 2 ? 1 : 0);
#pragma unroll 1
  for (int i = 0; i < passes; ++i) {
    SeriesPass ps;
    const bool draft = i < steps;
    if (draft) {
      // step 1 takes the token before the pending one along (see tsd_draft_propose)
      ps = i == 0 ? SeriesPass{2, len - 1, 0, X, 1, 2} : SeriesPass{1, len + i, i + 1, X + (long)i * P, 0, i + 2};
    } else {
      ps = SeriesPass{p.step_only ? 1 : Kr + 1, len, 1, p.mu_p + (long)b * p.mu_stride, 0, 0};
    }
    run_any_pass<RT>(p, p.m[draft ? 1 : 0], ps, series_lds, f, [&] {
      if (i + 1 < passes) prefetch_embed(p.m[i + 1 < steps ? 1 : 0], P, wave, tid & 63, f);
    });
  }
  if (!(p.phases & 4)) return;
  if (tid >= 256) return;  // (a barrier waits for the wavefronts that are left)
  const int2 now = accept_step(a);
  if (!c.host) return;
  __shared__ int last;
  if (tid == 0) {
    __hip_atomic_store(c.active + b, now.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(c.committed + b, now.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    last = __hip_atomic_fetch_add(c.ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
    if (last) __hip_atomic_store(c.ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (last) compact(c);
}

// The context of series blockIdx.x of the list through model blockIdx.y, 16 RT tokens at a time.
template <int RT>
__global__ __launch_bounds__(kThreads) void series_context_kernel(const SeriesP p, const float* znorm, int N) {
  extern __shared__ __attribute__((aligned(16))) float series_lds[];
  const int b = p.act ? p.act[blockIdx.x] : (int)blockIdx.x;
  const SeriesModel& m = p.m[blockIdx.y];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Frags f[2];
  prefetch_embed(m, p.P, wave, threadIdx.x & 63, f);
  const float* z = znorm + (long)b * N * p.P;
#pragma unroll 1
  for (int t0 = 0; t0 < N - 1; t0 += 16 * RT) {
    const int nq = min(16 * RT, N - 1 - t0);
    set_up<RT>(p, blockIdx.y, b, t0, nq, series_lds, [&](int t) { return z + (long)(t0 + t) * p.P; });
    run_any_pass<RT>(p, m, SeriesPass{nq, t0, 0, nullptr, 0, 0}, series_lds, f,
                     [&] { prefetch_embed(m, p.P, wave, threadIdx.x & 63, f); });
  }
}

namespace {

// The weights [N][K] in the order the products read them; qkv_hd > 0: columns in rotary-pair order within heads of qkv_hd.
__global__ __launch_bounds__(256) void series_pack_kernel(const float* src, float* dst, int N, int K, int runs, int qkv_hd) {
  const long total = (long)up16(N) * runs * 16;
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
    const int j = (int)(i & 3), lane = (int)((i >> 2) & 63);
    const long br = i >> 8;
    const int t = (int)(br % runs), blk = (int)(br / runs), l15 = lane & 15, k = t * 16 + j * 4 + (lane >> 4);
    int col = blk * 16 + l15;
    if (qkv_hd) {
      const int bph = qkv_hd >> 4, hs = blk / bph;
      col = hs * qkv_hd + (blk - hs * bph) * 8 + (l15 & 7) + (l15 < 8 ? 0 : qkv_hd >> 1);
    }
    dst[i] = k < K && col < N ? src[(long)col * K + k] : 0.f;
  }
}

int rows_of(int tokens) { return tokens <= 16 ? 16 : 32; }

constexpr size_t kMostLds = 156 * 1024;  // (the rest is the acceptance step's)

// LDS of a launch with passes of `rows` rows over `tokens` tokens
size_t lds_bytes(const tsd_config& c, int rows, int tokens, int models) {
  int shared = 0, D = 0, half = 0;
  for (const tsd_model_cfg* m : {&c.target, &c.draft}) {
    shared = std::max(shared, shared_words(m->d_model, m->d_ff, rows, c.max_tokens));
    D = std::max(D, m->d_model);
    half = std::max(half, m->d_model / m->n_heads / 2);
  }
  return (size_t)carve_of(D, half, c.patch, rows, tokens, models, c.max_tokens, shared).total * 4;
}

// Rows at a time of a context pass of so many tokens (0: it is none of this kernel's).
int context_rows(const tsd_config& c, int tokens) {
  for (int rows = rows_of(tokens); rows >= 16; rows -= 16)
    if (lds_bytes(c, rows, rows, 1) <= kMostLds) return rows;
  return 0;
}

}  // namespace

size_t series_packed_words(int N, int K) { return (size_t)up16(N) * up16(K); }

hipError_t launch_series_pack(const float* src, float* dst, int N, int K, int qkv_hd, hipStream_t st) {
  const size_t total = series_packed_words(N, K);
  hipLaunchKernelGGL(series_pack_kernel, dim3((unsigned)std::min<size_t>((total + 255) / 256, 4096)), dim3(256), 0, st, src, dst, N, K, up16(K) >> 4, qkv_hd);
  return hipGetLastError();
}

// Series of a decode that one round takes a workgroup each for, two for every compute unit.  Behind that the launches of the tiled path
// fill the chip: target-only steps gain no more, whole decodes still a little; rounds and steps have one limit, so that a batch's decode is
// one kind of pass.  (Decodes and target-only steps, us, kernel by kernel / this: 2 layers of 64, 512 series 673 and 471 / 309 and 292, 1024
// series 768 and 568 / 551 and 566; 3 layers of 128, 512 series 1143 and 981 / 677 and 895, 1024 series 1347 and 1243 / 1211 and 1764.  Up to
// 512 series, widths 32 to 128, 1 to 12 layers, 8 to 400 patches of context: decodes 1.3 to 3.6 times as fast, steps 1.06 to 4.9.)  The
// batch counts, not who is still active: the late rounds of a larger batch stay launch by launch.
constexpr int kMostSeries = 512;
bool series_round_ok(int n) { return n <= kMostSeries; }

bool series_rounds_ok(const tsd_config& c) {
  if (c.dtype != TSD_F32 || c.target.n_experts || c.draft.n_experts || (c.flags & (TSD_FLAG_SAMPLE_PROPOSALS | TSD_FLAG_NAIVE_VERIFY))) return false;
  for (const tsd_model_cfg* m : {&c.target, &c.draft})
    if (shape_of(m->d_model, m->n_heads, m->d_ff) < 0) return false;
  return lds_bytes(c, rows_of(c.K + 1), c.K + 2, 2) <= kMostLds;
}

int series_shape(const tsd_model_cfg& m) { return shape_of(m.d_model, m.n_heads, m.d_ff); }
bool series_context_ok(const tsd_config& c, int n, int tokens) {
  return series_context_pays(std::max(c.target.d_model, c.draft.d_model), n, tokens) && context_rows(c, tokens) > 0;
}

hipError_t prepare_series() {
  const void* fns[4] = {reinterpret_cast<const void*>(&series_round_kernel<1>), reinterpret_cast<const void*>(&series_round_kernel<2>),
                        reinterpret_cast<const void*>(&series_context_kernel<1>), reinterpret_cast<const void*>(&series_context_kernel<2>)};
  for (const void* f : fns) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMostLds);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_series_round(const tsd_config& c, SeriesP p, const AcceptP& a, const CompactP& k, hipStream_t st) {
  const int rows = rows_of(std::max(2, p.step_only ? 1 : p.K + 1));
  p.tokens = p.K + 2;
  p.models = 2;
  const size_t smem = lds_bytes(c, rows, p.tokens, 2);
  if (smem > kMostLds) return hipErrorInvalidValue;
  if (rows == 16) hipLaunchKernelGGL(series_round_kernel<1>, dim3(p.n), dim3(kThreads), smem, st, p, a, k);
  else hipLaunchKernelGGL(series_round_kernel<2>, dim3(p.n), dim3(kThreads), smem, st, p, a, k);
  return hipGetLastError();
}

hipError_t launch_series_context(const tsd_config& c, SeriesP p, const float* znorm, int N, hipStream_t st) {
  const int rows = context_rows(c, N - 1);
  if (!rows) return hipErrorInvalidValue;
  p.tokens = rows;
  p.models = 1;
  const size_t smem = lds_bytes(c, rows, rows, 1);
  if (rows == 16) hipLaunchKernelGGL(series_context_kernel<1>, dim3(p.n, 2), dim3(kThreads), smem, st, p, znorm, N);
  else hipLaunchKernelGGL(series_context_kernel<2>, dim3(p.n, 2), dim3(kThreads), smem, st, p, znorm, N);
  return hipGetLastError();
}

}  // namespace tsd
