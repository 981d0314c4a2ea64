// Decode passes of at most 32 rows (one series up to a few: the latency regime) as one resident kernel: all draft steps
// of a round and the verification pass, layer by layer, without leaving the GPU.
//
// Such a pass is a chain of products that each stream a few MB of weights past a handful of rows.  Kernel by kernel every
// link of the chain costs 6 us (dispatch, first loads, last stores), whatever it does: a round of one series through 24 layers
// of 1024 (draft 2 x 256, K = 4) is 170 launches and 1.05 ms for 0.6 GB of weights.  Here one workgroup per compute unit
// stays for the whole chain and the links are joined by flags: the workgroups of a stage publish their results and raise
// their flag, those of the next stage watch the flags.  The hop alone costs 1.7 us at 256 workgroups (measured: one flag
// per 64-byte line, every workgroup polling all of them; one shared counter takes 4.1 us, flags packed into few lines 3.7).
// That round now takes 0.71 ms, one of five series through 8 layers of 512 0.39 instead of 0.52; a stage is 1.1-1.7 us of
// hop, 1.2-1.6 of operands and products and 0.9 of epilogue and write-through.
//
//   * A workgroup owns a fixed few columns (4, 8 or 16) of every product, the fewest with which the product still fits
//     the 256 workgroups.  The weights of its next product depend on nothing, so their loads are issued as soon as the
//     registers are free, before the hop: they arrive while the flags are being watched.
//   * Four worker wavefronts split the product's k range; a fifth, the control wavefront, adds their partial sums,
//     runs the epilogue, publishes, raises the flag and watches the others'.  (It issues no weight loads, which would
//     hold up its polls: loads return in order.)
//   * The columns of the residual stream a workgroup owns are the same for the embedding, the attention output and the FFN
//     down product: its fp32 residual never leaves LDS, only the bf16 shadow the next products read does.
//   * Attention: one (series, head) per workgroup; the keys of earlier passes are fetched before the hop.
//   * What workgroups hand each other is written through to memory (agent scope, "sc1") at an address nobody has read in
//     this launch, so no cache is written back or invalidated at a hop (see the exchange buffer below).
//   * Every sum is formed in the order of the kernels this replaces (gemm_skinny.hip, attn_mfma.h): same bits.
//
// All workgroups of a launch have to be resident together: one per compute unit, and a process has one launch of this kernel
// on a device at a time (launch_small_round).  Other processes are not seen: where two launches have taken each other's compute units,
// neither can go on.  So every wait is bounded: a workgroup that has waited since its start for p.wait_ticks, or sees that another
// gave up, leaves, and the kernel behind the launch does its work (series_alone).
#include <algorithm>
#include <atomic>
#include <chrono>
#include <mutex>
#include <vector>

#include "accept_step.h"
#include "gemm_epilogue.h"
#include "tsd_internal.h"

namespace tsd {

namespace {

constexpr int kWg = kSmallRoundWorkgroups;
constexpr int kWorkers = kSmallRoundWorkers;
constexpr int kThreads = (kWorkers + 1) * 64;
constexpr int kRowsMax = kSmallRoundRows;
constexpr int kFlagWords = kSmallRoundFlagWords;  // one flag per 64-byte line
constexpr int kLdp = 18;                          // columns of a partial-sum row in LDS (padded)
constexpr int kSc1 = 16;                          // cache policy of the exchange: agent scope

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
using Rsrc = __amdgpu_buffer_rsrc_t;

__device__ __forceinline__ Rsrc rsrc_of(const void* p, long bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ u32x4 load16(Rsrc r, int off) { return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kSc1); }
__device__ __forceinline__ void publish4(void* p, unsigned v) {
  __hip_atomic_store(reinterpret_cast<unsigned*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish_bf16x2(bf16* p, float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 v = {(bf16)a, (bf16)b};
  publish4(p, __builtin_bit_cast(unsigned, v));
}

// Everything between two hops is executed by a handful of wavefronts one after the other, so its duration is the number of
// instructions on the way (a first version with divisions, clamps and selects on the way took 3.4 us per product for 0.9 us
// of loads): what depends on sizes alone comes from the host (SmallProd), what depends on the pass is formed once per pass.

// Column `c` (0 .. cw - 1) of workgroup `unit`.
template <bool QKV>
__device__ __forceinline__ int column_of(const SmallProd& d, int unit, int c) {
  if (!QKV) return (unit << d.cs) + c;
  const int half = 1 << (d.cs - 1), head = unit >> (6 - d.cs), j = unit & ((64 >> d.cs) - 1);  // heads of q, then k, then v are consecutive
  return head * 64 + j * half + (c < half ? c : 32 + c - half);
}

// A worker's weights of one product: at most eight 16-byte pieces per lane.  A worker takes four slabs.  With fewer than 16
// columns the 16 lane columns of an MFMA operand hold several slabs side by side: piece i of k-step j of the slabs,
// lane column li: column li % cw of slab 4 wave + (16 / cw) i + li / cw.  Pieces are numbered j * (cw / 4) + i.
struct Weights {
  bf16x8 f[8];
};

template <int CW>
__device__ __forceinline__ void load_weights(const bf16* W, unsigned off, int per, Weights& w) {
  constexpr int PB = CW / 4, SB = 16 / CW;
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const int j = t / PB, i = t % PB;
    if (j < per) w.f[t] = *reinterpret_cast<const bf16x8*>(W + (slab_start(SB * i, per) + j * 32) + off);
  }
}

// Starts the loads of this worker's share of the workgroup's weights of a product, W its matrix.
template <bool QKV>
__device__ __forceinline__ void prefetch(const SmallProd& d, const bf16* W, int wg, int wave, int lane, Weights& w) {
  if (wg >= d.units || 4 * wave >= d.used) return;
  asm volatile("" : "+v"(lane));  // (an opaque copy: keeps the address arithmetic below from being hoisted to the kernel's top)
  const int li = lane & 15, col = column_of<QKV>(d, wg, li & ((1 << d.cs) - 1));
  const unsigned off = (unsigned)(col * d.K + slab_start(4 * wave + (li >> d.cs), d.per) + (lane >> 4) * 8);
  if (d.cs == 2) load_weights<4>(W, off, d.per, w);
  else if (d.cs == 3) load_weights<8>(W, off, d.per, w);
  else load_weights<16>(W, off, d.per, w);
}

// The embedding's k range may end inside a k-step or a slab: clamped reads, against zero activations.
__device__ __forceinline__ void prefetch_embed(const SmallProd& d, const bf16* W, int wg, int wave, int lane, Weights& w) {
  if (wg >= d.units || 4 * wave >= d.used) return;
  asm volatile("" : "+v"(lane));
  const int li = lane & 15, k0 = (4 * wave + (li >> 2)) * d.per * 32 + (lane >> 4) * 8;
  const bf16* row = W + (wg * 4 + (li & 3)) * d.K;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (j < d.per) w.f[j] = *reinterpret_cast<const bf16x8*>(row + min(k0 + j * 32, d.K - 8));
}

__device__ __forceinline__ void split_hi_lo(const float* f, bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    hi[e] = (bf16)f[e];
    lo[e] = (bf16)(f[e] - (float)hi[e]);
  }
}

struct Shared {
  union {
    struct {
      float part[16][kRowsMax][kLdp];  // by slab
      float ss[16][kRowsMax];
    } g;
    struct {
      bf16 vt[kWorkers][32 * 64];  // V rows on their way to the transposing read
      bf16 pf[kWorkers][64][8];    // exponentials, as operand fragments
      float psum[kWorkers][64], mx[kWorkers][16], m[kWorkers][16], alpha[kWorkers][16];
    } a;
  } u;
  float xown[kRowsMax][16];  // fp32 residual of the columns this workgroup owns
  int ser[kRowsMax], pos[kRowsMax], page[kRowsMax];
  int quit;
};

// One worker's share of a product of bf16 activations, R row slots (4, 8 or 16) per tile and NT tiles, CW columns.
// Like the weights, the rows of a pass with few of them share the 16 lane rows of an MFMA operand: lane row li of piece i
// holds row li % R of slab 4 wave + (16 / R) i + li / R.  An MFMA of such pieces is right where its row's and its column's
// slab agree, which is all that is kept.  No lane then fetches what another one has fetched already: 5 rows cost half the
// loads of 16, 4 columns a quarter.
template <int R, int NT, int CW>
__device__ __forceinline__ void product_t(const bf16* A, int K, int per, int M, bool norm, int wave, int lane, const Weights& w, Shared& sh) {
  asm volatile("" : "+v"(lane));
  constexpr int SA = 16 / R, SB = 16 / CW, G = SA < SB ? SA : SB, NACC = 4 / G, PA = R / 4, PB = CW / 4;
  const int li = lane & 15, lg = lane >> 4;
  unsigned row[NT];  // element offsets from A (uniform base, 32-bit offset: one address register per load)
#pragma unroll
  for (int r = 0; r < NT; ++r) row[r] = (unsigned)(min(r * 16 + li % R, M - 1) * K + slab_start(4 * wave + li / R, per) + lg * 8);
  f32x4 acc[NT][NACC];  // g: slabs 4 wave + g G .. + G - 1
  float ss[NT][PA];
#pragma unroll
  for (int r = 0; r < NT; ++r) {
#pragma unroll
    for (int i = 0; i < PA; ++i) ss[r][i] = 0.f;
#pragma unroll
    for (int c = 0; c < NACC; ++c) acc[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  constexpr int JMAX = 8 / PB;                                       // k-steps of a slab whose weights fit the eight pieces
  constexpr int JC = JMAX * NT * PA <= 16 ? JMAX : 16 / (NT * PA);  // k-steps whose rows are in registers at a time
#pragma unroll
  for (int j0 = 0; j0 < JMAX; j0 += JC) {
    if (j0 >= per) break;
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 a[JC][NT][PA];
#pragma unroll
    for (int j = 0; j < JC; ++j) {
      if (j0 + j >= per) break;
#pragma unroll
      for (int r = 0; r < NT; ++r)
#pragma unroll
        for (int i = 0; i < PA; ++i) a[j][r][i] = *reinterpret_cast<const bf16x8*>(A + (slab_start(SA * i, per) + (j0 + j) * 32) + row[r]);
    }
#pragma unroll
    for (int j = 0; j < JC; ++j) {
      if (j0 + j >= per) break;
#pragma unroll
      for (int r = 0; r < NT; ++r) {
        if (norm) {
#pragma unroll
          for (int i = 0; i < PA; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float f = (float)a[j][r][i][e];
              ss[r][i] = fmaf(f, f, ss[r][i]);
            }
        }
#pragma unroll
        for (int g = 0; g < NACC; ++g)
          acc[r][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j][r][g * G / SA], w.f[(j0 + j) * PB + g * G / SB], acc[r][g], 0, 0, 0);
      }
    }
  }
  // this lane's accumulator elements are rows 4 lg + i, column li of the operand tile
  const int sA = 4 * lg / R, sB = li / CW;
  float* part = &sh.u.g.part[4 * wave][4 * lg % R][li % CW];
#pragma unroll
  for (int g = 0; g < NACC; ++g) {
    const int s = sB - (g * G) % SB;
    if (s >= 0 && s < G && s == sA - (g * G) % SA) {
      float* to = part + (g * G + s) * (kRowsMax * kLdp);
#pragma unroll
      for (int r = 0; r < NT; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) to[(r * 16 + i) * kLdp] = acc[r][g][i];
    }
  }
  if (norm) {
#pragma unroll
    for (int r = 0; r < NT; ++r)
#pragma unroll
      for (int i = 0; i < PA; ++i) {
        float s = ss[r][i];
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        if (lg == 0) sh.u.g.ss[4 * wave + SA * i + li / R][r * 16 + li % R] = s;
      }
  }
}

template <int R, int NT>
__device__ __forceinline__ void product_cw(const SmallProd& d, const bf16* A, int M, bool norm, int wave, int lane, const Weights& w, Shared& sh) {
  if (d.cs == 2) product_t<R, NT, 4>(A, d.K, d.per, M, norm, wave, lane, w, sh);
  else if (d.cs == 3) product_t<R, NT, 8>(A, d.K, d.per, M, norm, wave, lane, w, sh);
  else product_t<R, NT, 16>(A, d.K, d.per, M, norm, wave, lane, w, sh);
}

__device__ __forceinline__ void product(const SmallProd& d, const bf16* A, int M, bool norm, int wave, int lane, const Weights& w, Shared& sh) {
  if (4 * wave >= d.used) return;
  if (M <= 4) product_cw<4, 1>(d, A, M, norm, wave, lane, w, sh);
  else if (M <= 8) product_cw<8, 1>(d, A, M, norm, wave, lane, w, sh);
  else if (M <= 16) product_cw<16, 1>(d, A, M, norm, wave, lane, w, sh);
  else product_cw<16, 2>(d, A, M, norm, wave, lane, w, sh);
}

// The same for fp32 rows, split into hi + lo bf16 parts (patches, and the residual the head reads): row r's values at
// src(r, k), rows not shared between slabs, four columns, slabs of at most four k-steps.
template <bool NORM, typename Src>
__device__ __forceinline__ void product_f32(const SmallProd& d, int M, int wave, int lane, const Weights& w, Shared& sh, Src src) {
  asm volatile("" : "+v"(lane));
  if (4 * wave >= d.used) return;
  const int K = d.K, per = d.per, li = lane & 15, lg = lane >> 4;
  const bool ragged = d.used * per * 32 != K;
#pragma unroll 1
  for (int r = 0; r < 2; ++r) {
    if (r * 16 >= M) break;
    const int row = min(r * 16 + li, M - 1);
    f32x4 acc[4];
    float ss[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
      ss[s] = 0.f;
    }
    auto two = [&](auto first) {  // k-steps j0 and j0 + 1 of all four slabs
      constexpr int j0 = decltype(first)::value;
      float f[4][2][8];
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int j = 0; j < 2; ++j) src(row, min(((4 * wave + s) * per + min(j0 + j, per - 1)) * 32 + lg * 8, K - 8), f[s][j]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (j0 + j >= per) break;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          bf16x8 b = w.f[j0 + j];  // (lane columns with li / 4 == s are slab s's: the others' products are dropped)
          if (ragged && ((4 * wave + s) * per + j0 + j) * 32 + lg * 8 >= K) {
            b = bf16x8{};
#pragma unroll
            for (int e = 0; e < 8; ++e) f[s][j][e] = 0.f;
          }
          bf16x8 hi, lo;
          split_hi_lo(f[s][j], hi, lo);
          if constexpr (NORM) {
#pragma unroll
            for (int e = 0; e < 8; ++e) ss[s] = fmaf(f[s][j][e], f[s][j][e], ss[s]);
          }
          acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, b, acc[s], 0, 0, 0);
          acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, b, acc[s], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    two(std::integral_constant<int, 0>{});
    if (per > 2) two(std::integral_constant<int, 2>{});
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if ((li >> 2) == s) {
#pragma unroll
        for (int i = 0; i < 4; ++i) sh.u.g.part[4 * wave + s][r * 16 + lg * 4 + i][li & 3] = acc[s][i];
      }
      if constexpr (NORM) {
        float t = ss[s];
        t += __shfl_xor(t, 16);
        t += __shfl_xor(t, 32);
        if (lg == 0) sh.u.g.ss[4 * wave + s][r * 16 + li] = t;
      }
    }
  }
}

// Control wavefront: columns c, c + 1 of a row's partial sums and its partial row sums, four slabs at a time: their reads
// together, then the additions in slab order.  (Sixteen are usual, four for short k ranges; others are a multiple of one.)
struct Sums {
  float2 a, b;  // the columns, and their rotary partners
  float ss;     // row sum of squares
};
template <bool PARTNER, bool ROWS>
__device__ __forceinline__ Sums sums_of(const Shared& sh, int row, int c, int partner, int used) {
  Sums s{make_float2(0.f, 0.f), make_float2(0.f, 0.f), 0.f};
  const float *pa = &sh.u.g.part[0][row][c], *pb = &sh.u.g.part[0][row][partner], *pr = &sh.u.g.ss[0][row];
  auto chunk = [&](int w0, auto count) {
    constexpr int N = decltype(count)::value;
    float2 va[N], vb[N];
    float vr[N];
#pragma unroll
    for (int w = 0; w < N; ++w) {
      va[w] = *reinterpret_cast<const float2*>(pa + (w0 + w) * (kRowsMax * kLdp));
      if constexpr (PARTNER) vb[w] = *reinterpret_cast<const float2*>(pb + (w0 + w) * (kRowsMax * kLdp));
      if constexpr (ROWS) vr[w] = pr[(w0 + w) * kRowsMax];
    }
#pragma unroll
    for (int w = 0; w < N; ++w) {
      s.a.x += va[w].x;
      s.a.y += va[w].y;
      if constexpr (PARTNER) {
        s.b.x += vb[w].x;
        s.b.y += vb[w].y;
      }
      if constexpr (ROWS) s.ss += vr[w];
    }
  };
  if (used == 16) {
    chunk(0, std::integral_constant<int, 16>{});
  } else {
    int w = 0;
    for (; w + 4 <= used; w += 4) chunk(w, std::integral_constant<int, 4>{});
    for (; w < used; ++w) chunk(w, std::integral_constant<int, 1>{});
  }
  return s;
}
__device__ __forceinline__ float norm_scale(float ss, int K) { return rsqrtf(ss / (float)K + kRmsEps); }

// Attention of one (series, head) by the four workers, 32-key steps as in attn_mfma.h: the same operations on the same values
// in the same order, hence the same bits.  Only the running sums are a chain over the steps; so, per trip of four steps:
//   worker t: scores of step t, their maxima                                          (barrier)
//   worker t: running maximum before and at its step, exponentials, rescale factor    (barrier)
//   worker b: output dims 16 b .. 16 b + 15 through the trip's steps in order.
// The rows of a step of keys cached before this pass (all below `base`) are fetched before `ready()`, the hop.
template <typename Ready>
__device__ __forceinline__ bool attend(const SmallRoundP& p, const bf16* pool, const bf16* Q, bf16* out, int ld, int h, int Hh, int my_page,
                                       int base, int nq, int wave, int lane, Shared& sh, Ready ready) {
  asm volatile("" : "+v"(lane));
  const int qi = lane & 15, g = lane >> 4;
  const int PT = p.PT, pts = p.pt_shift;
  const int page_elems = 2 * Hh * PT * 64, v_off = Hh * PT * 64;
  const int total = base + nq, qrow = min(qi, nq - 1), qpos = base + qrow;
  bf16x8 kf[2][2], vf[4], qf[2];
  auto fetch = [&](int sb) {
#pragma unroll
    for (int bi = 0; bi < 2; ++bi) {
      const int key = min(sb + 8 * (qi >> 2) + 4 * bi + (qi & 3), total - 1);
      const int page = __shfl(my_page, key >> pts);
      const bf16* kp = pool + (long)page * page_elems + ((h * PT + (key & (PT - 1))) * 64 + g * 8);
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) kf[bi][kk] = *reinterpret_cast<const bf16x8*>(kp + kk * 32);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int key = min(sb + (lane >> 3) + 8 * i, total - 1);
      const int page = __shfl(my_page, key >> pts);
      vf[i] = *reinterpret_cast<const bf16x8*>(pool + (long)page * page_elems + (v_off + (h * PT + (key & (PT - 1))) * 64 + (lane & 7) * 8));
    }
  };
  const bool early = wave * 32 + 32 <= base;
  if (early) fetch(wave * 32);
  if (!ready()) return false;
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(Q + (qrow * ld + kk * 32 + g * 8));
  f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;  // of query qi, before the trip
  for (int s0 = 0; s0 < total; s0 += 32 * kWorkers) {
    const int sb = s0 + wave * 32;
    const int steps = min(kWorkers, (total - s0 + 31) >> 5);  // of this trip
    float sv[8];
    if (s0) lds_barrier();  // the previous trip's reads are done
    if (sb < total) {
      if (s0 || !early) fetch(sb);
      f32x4 sc[2];
#pragma unroll
      for (int bi = 0; bi < 2; ++bi) {
        sc[bi] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) sc[bi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[bi][kk], qf[kk], sc[bi], 0, 0, 0);
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) sv[j] = sc[j >> 2][j & 3] * p.scale;
      if (sb + 31 > base) {  // some of the keys may lie past a query
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (sb + 8 * g + j > qpos) sv[j] = -INFINITY;
      }
      float mx = sv[0];
#pragma unroll
      for (int j = 1; j < 8; ++j) mx = fmaxf(mx, sv[j]);
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      if (g == 0) sh.u.a.mx[wave][qi] = mx;
      if (sb + 32 > total) {  // past the cache's end anything may lie: zero rows
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (sb + (lane >> 3) + 8 * i >= total) vf[i] = bf16x8{};
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<bf16x8*>(sh.u.a.vt[wave] + ((lane >> 3) + 8 * i) * 64 + (((lane & 7) * 8 + 16 * i) & 63)) = vf[i];
    }
    lds_barrier();
    if (sb < total) {
      float m_old = m_run;
#pragma unroll
      for (int t = 0; t < kWorkers - 1; ++t)
        if (t < wave) m_old = fmaxf(m_old, sh.u.a.mx[t][qi]);
      const float m_new = fmaxf(m_old, sh.u.a.mx[wave][qi]);  // finite: key 0 is visible to every query
      bf16x8 pf;
      float psum = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float e = __expf(sv[j] - m_new);
        psum += e;
        pf[j] = (bf16)e;
      }
      *reinterpret_cast<bf16x8*>(sh.u.a.pf[wave][lane]) = pf;
      sh.u.a.psum[wave][lane] = psum;
      if (g == 0) {
        sh.u.a.alpha[wave][qi] = __expf(m_old - m_new);
        sh.u.a.m[wave][qi] = m_new;
      }
    }
    lds_barrier();
    typedef short short4v __attribute__((ext_vector_type(4)));
    typedef short short8v __attribute__((ext_vector_type(8)));
#pragma unroll
    for (int t = 0; t < kWorkers; ++t) {
      if (t >= steps) break;
      short4v hv[2];
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const bf16* src = sh.u.a.vt[t] + (8 * g + 4 * half + (qi >> 2)) * 64 + ((wave * 16 + 4 * (qi & 3) + 16 * g) & 63);
        hv[half] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)src);
      }
      const short8v both = __builtin_shufflevector(hv[0], hv[1], 0, 1, 2, 3, 4, 5, 6, 7);
      const bf16x8 pt = *reinterpret_cast<const bf16x8*>(sh.u.a.pf[t][lane]);
      l_run = l_run * sh.u.a.alpha[t][qi] + sh.u.a.psum[t][lane];
      const float4 ar = *reinterpret_cast<const float4*>(&sh.u.a.alpha[t][4 * g]);
      o[0] *= ar.x;
      o[1] *= ar.y;
      o[2] *= ar.z;
      o[3] *= ar.w;
      o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pt, __builtin_bit_cast(bf16x8, both), o, 0, 0, 0);
    }
    m_run = sh.u.a.m[steps - 1][qi];
  }
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
  const float inv = 1.f / l_run;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (r >= nq) break;  // (uniform: rows r, r + 4, .. of the tile)
    const float v = o[r] * __shfl(inv, 4 * g + r), v2 = __shfl_xor(v, 1);
    const int qq = 4 * g + r;
    if (qq < nq && !(qi & 1)) publish_bf16x2(out + (qq * ld + wave * 16 + qi), v, v2);
  }
  return true;
}

// Barriers of attend() after the hop, for the control wavefront to take part in.
__device__ __forceinline__ void attend_barriers(int total) {
  for (int s0 = 0; s0 < total; s0 += 32 * kWorkers) {
    if (s0) lds_barrier();
    lds_barrier();
    lds_barrier();
  }
}

// The stages of a pass in order, as both kinds of wavefront walk them; `ep` and `units` say what the next hop waits for.
struct Walk {
  unsigned ep;  // value the flags of the previous stage's workgroups reach
  int units;    // workgroups of the previous stage (0: the inputs come from before the launch)
  __device__ __forceinline__ void done(int u) {
    ++ep;
    units = u;
  }
};

// The exchange buffer: what workgroups hand each other, at a fresh address for every stage of a launch.  No cache can hold
// an older copy of such a line (caches start a launch empty of it), so the readers use ordinary loads and the 32 workgroups
// of an XCD share one fetch through their L2; only the stores have to go through to memory.  (Reading reused buffers past
// the caches: 6.7 us per FFN down stage for one series through 4096 x 1024, most of it 256 workgroups fetching 40 KB each
// from the last-level cache.)
// (Its layout: small_round_plan.h.)

enum Kind { kQkv, kAttend, kOut, kUp, kDown };

// What both kinds of wavefront derive from the arguments, per pass.
struct PassView {
  const SmallModel* m;
  bool draft;
  int step, nq, M, D;
  char* x;  // this pass's part of the exchange buffer
  __device__ __forceinline__ PassView(const SmallRoundP& p, int ps, int Kd, int Kr, int n)
      : m(&p.m[ps < Kd ? 1 : 0]), draft(ps < Kd), step(ps + 1), nq(ps < Kd ? (ps == 0 ? 2 : 1) : Kr + 1) {
    M = n * nq;
    D = m->D;
    x = reinterpret_cast<char*>(p.exchange) + (size_t)(draft ? ps : p.k_max) * p.m[1].pass_bytes;
  }
  // rows entering layer l, its queries, attention output, rows between the two halves, hidden rows; residual for the head
  __device__ __forceinline__ bf16* rows(int l, int which) const {
    return reinterpret_cast<bf16*>(x + (size_t)l * m->slab_bytes + small_part_offset(D, which));
  }
  __device__ __forceinline__ float* residual() const { return reinterpret_cast<float*>(x + (size_t)m->L * m->slab_bytes); }
  __device__ __forceinline__ const bf16* weights(const SmallProd& d, int l) const {
    return reinterpret_cast<const bf16*>(reinterpret_cast<const char*>(d.W) + (size_t)l * m->wstride);
  }
};

// Rows of a pass: series, position and cache page of each (between two barriers, by the first 32 lanes).
__device__ __forceinline__ void set_rows(const SmallRoundP& p, const PassView& v, Shared& sh) {
  const int tid = threadIdx.x;
  if (tid < kRowsMax) {
    const int r = min(tid, v.M - 1), sl = r / v.nq, t = r - sl * v.nq;
    const int b = p.act ? p.act[sl] : sl;
    const int pos = p.len[b] + (v.draft ? (v.step == 1 ? t - 1 : v.step - 1) : t);
    sh.ser[tid] = b;
    sh.pos[tid] = pos;
    sh.page[tid] = p.page_table[(long)b * p.pt_stride + (pos >> p.pt_shift)];
  }
}

// Eight values of a row's patch, from value k on.  (Patches are exchanged through reused lines: read past the caches; all three
// arrays lie behind `pending`.)
__device__ __forceinline__ Rsrc patches_of(const SmallRoundP& p) { return rsrc_of(p.pending, 0x7fffffff); }
__device__ __forceinline__ void load_patch(const SmallRoundP& p, const PassView& v, const Shared& sh, Rsrc patches, int r, int k, float* f) {
  const int P = p.P, sl = r / v.nq, t = r - sl * v.nq;
  const long b = sh.ser[r];
  const float* src;
  if (v.draft)
    src = v.step == 1 ? (t == 0 ? p.prev : p.pending) + b * P : p.X + b * p.x_stride + (long)(v.step - 2) * P;
  else
    src = t == 0 ? p.pending + b * P : p.X + b * p.x_stride + (long)(t - 1) * P;
  const int off = (int)(reinterpret_cast<const char*>(src + k) - reinterpret_cast<const char*>(p.pending));
  *reinterpret_cast<u32x4*>(f) = load16(patches, off);
  *reinterpret_cast<u32x4*>(f + 4) = load16(patches, off + 16);
}

// Column pairs of a product's columns, one after the other along the rows, over the lanes of a wavefront.
template <typename Fn>
__device__ __forceinline__ void each_pair(const SmallProd& d, int M, int lane, Fn fn) {
  const int sft = d.cs - 1;
  for (int i = lane; i < M << sft; i += 64) {
    const int row = i >> sft;
    fn(row, (i & ((1 << sft) - 1)) * 2);
  }
}

// Epilogues that need nothing but the partial sums: FFN up with GELU, and the head.
__device__ __forceinline__ void finish_up(const SmallModel& m, const PassView& v, bf16* hidden, int wg, int lane, const Shared& sh) {
  const SmallProd& d = m.up;
  bf16* hid = hidden + (wg << d.cs);
  each_pair(d, v.M, lane, [&](int row, int c) {
    const Sums z = sums_of<false, true>(sh, row, c, 0, d.used);
    const float2 s = z.a;
    const float rs = norm_scale(z.ss, v.D);
    publish_bf16x2(hid + row * m.F + c, gelu_tanh(s.x * rs), gelu_tanh(s.y * rs));
  });
}
__device__ __forceinline__ void finish_head(const SmallRoundP& p, const SmallModel& m, const PassView& v, int wg, int lane, const Shared& sh) {
  const SmallProd& d = m.head;
  const int P = p.P;
  each_pair(d, v.M, lane, [&](int row, int c) {
    const int sl = row / v.nq, t = row - sl * v.nq, col = (wg << d.cs) + c;
    const Sums z = sums_of<false, true>(sh, row, c, 0, d.used);
    const float rs = norm_scale(z.ss, v.D);
    float2 s = z.a;
    s.x *= rs;
    s.y *= rs;
    const long b = sh.ser[row];
    if (!v.draft) {
      *reinterpret_cast<float2*>(p.mu_p + b * p.mu_stride + (long)t * P + col) = s;
    } else if (t == v.nq - 1) {  // (step 1 emits from the pending token only)
      float* x = p.X + b * p.x_stride + (long)(v.step - 1) * P + col;
      publish4(x, __builtin_bit_cast(unsigned, s.x));
      publish4(x + 1, __builtin_bit_cast(unsigned, s.y));
    }
  });
}

// The stage's results are published.
__device__ __forceinline__ void raise_flag(const SmallRoundP& p, int wg, int lane, unsigned value) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (lane == 0) __hip_atomic_store(p.flags + wg * kFlagWords, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void give_up(const SmallRoundP& p) {
  __hip_atomic_store(p.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(p.host_status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ bool hop_worker(Shared& sh) {
  lds_barrier();
  return *reinterpret_cast<volatile int*>(&sh.quit) == 0;
}

__device__ __forceinline__ void worker_loop(const SmallRoundP& p, int n, int Kr, int Kd, int n_pass, int wave, int lane, Shared& sh) {
  const int wg = blockIdx.x;
  Weights w;
  {
    const PassView v(p, 0, Kd, Kr, n);
    prefetch_embed(v.m->embed, v.m->embed.W, wg, wave, lane, w);
  }
  for (int ps = 0; ps < n_pass; ++ps) {
    const PassView v(p, ps, Kd, Kr, n);
    const SmallModel& m = *v.m;
    const int D = v.D, M = v.M, nq = v.nq, tasks = n * m.Hh;
    const Rsrc patches = patches_of(p);
    lds_barrier();  // (the previous pass's rows are no longer read)
    set_rows(p, v, sh);
    lds_barrier();
    // this workgroup's (series slot, head)
    int head = 0, r0 = 0, base = 0, my_page = 0;
    if (wg < tasks) {
      const int sl = wg / m.Hh;
      head = wg - sl * m.Hh;
      r0 = sl * nq;
      base = __builtin_amdgcn_readfirstlane(sh.pos[r0]);
      my_page = p.page_table[(long)sh.ser[r0] * p.pt_stride + min(lane, p.pt_stride - 1)];
    }

    if (wg < m.embed.units) {
      if (!hop_worker(sh)) return;
      product_f32<false>(m.embed, M, wave, lane, w, sh, [&](int r, int k, float* f) { load_patch(p, v, sh, patches, r, k, f); });
      lds_barrier();
    }
    // (after the barrier: the control wavefront does not wait for the loads to be issued)
    prefetch<true>(m.qkv, m.qkv.W, wg, wave, lane, w);

    for (int l = 0; l < m.L; ++l) {
      // One body for the products of a layer (written out four times they crowd the instruction cache and the scalar registers),
      // attention behind the first.
#pragma unroll 1
      for (int kind = kQkv; kind <= kDown; ++kind) {
        if (kind == kAttend) {
          if (wg >= tasks) continue;
          if (!attend(p, m.kv_pool + (size_t)l * m.layer_pool_elems, v.rows(l, kQuery) + r0 * D + head * 64, v.rows(l, kMixed) + r0 * D + head * 64,
                      D, head, m.Hh, my_page, base, nq, wave, lane, sh, [&] { return hop_worker(sh); }))
            return;
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          lds_barrier();
          continue;
        }
        const SmallProd& d = kind == kQkv ? m.qkv : kind == kOut ? m.out : kind == kUp ? m.up : m.down;
        if (wg < d.units) {
          if (!hop_worker(sh)) return;
          product(d, v.rows(l, kind == kQkv ? kIn : kind == kOut ? kMixed : kind == kUp ? kMid : kHidden), M, kind == kQkv || kind == kUp,
                  wave, lane, w, sh);
          lds_barrier();
          // (768 clocks later: issued at once, 8 MB of weights stand in front of the few KB the control wavefront publishes
          //  next)
          __builtin_amdgcn_s_sleep(12);
        }
        // the weights of the workgroup's next product
        if (kind == kDown && l + 1 < m.L) {
          prefetch<true>(m.qkv, v.weights(m.qkv, l + 1), wg, wave, lane, w);
        } else {
          const SmallProd& nx = kind == kQkv ? m.out : kind == kOut ? m.up : kind == kUp ? m.down : m.head;
          prefetch<false>(nx, kind == kDown ? nx.W : v.weights(nx, l), wg, wave, lane, w);
        }
      }
    }

    const bool more = ps + 1 < n_pass;
    if (wg < m.head.units) {
      if (!hop_worker(sh)) return;
      const float* xf = v.residual();
      product_f32<true>(m.head, M, wave, lane, w, sh, [&](int r, int k, float* f) {
        *reinterpret_cast<float4*>(f) = *reinterpret_cast<const float4*>(xf + (r * D + k));
        *reinterpret_cast<float4*>(f + 4) = *reinterpret_cast<const float4*>(xf + (r * D + k + 4));
      });
      lds_barrier();
    }
    if (more) {
      const SmallModel& nm = p.m[ps + 1 < Kd ? 1 : 0];
      prefetch_embed(nm.embed, nm.embed.W, wg, wave, lane, w);
    }
  }
}

__device__ __forceinline__ void control_loop(const SmallRoundP& p, int n, int Kr, int Kd, int n_pass, int lane, Shared& sh) {
  const int wg = blockIdx.x;
  const long long deadline = wall_clock64() + p.wait_ticks;
  Walk walk{p.epoch, 0};
  // The previous stage's results are there (false: give up); the workers are let go.
  auto hop = [&]() -> bool {
    bool go = true;
    if (walk.units) {
      const unsigned* f[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = p.flags + min(lane + 64 * j, walk.units - 1) * kFlagWords;
      for (int spin = 1;; ++spin) {
        unsigned x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = __hip_atomic_load(f[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bool ok = true;
#pragma unroll
        for (int j = 0; j < 4; ++j) ok = ok && small_flag_reached(x[j], walk.ep);
        if (__all(ok)) break;
        if ((spin & 63) == 0) {
          const int gone = __hip_atomic_load(p.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (gone || wall_clock64() > deadline) {
            if (lane == 0) {
              give_up(p);
              sh.quit = 1;
            }
            go = false;
            break;
          }
        }
      }
    }
    lds_barrier();
    return go;
  };
  auto raise = [&]() { raise_flag(p, wg, lane, walk.ep + 1); };

  for (int ps = 0; ps < n_pass; ++ps) {
    const PassView v(p, ps, Kd, Kr, n);
    const SmallModel& m = *v.m;
    const int D = v.D, Hh = m.Hh, M = v.M, nq = v.nq;
    lds_barrier();
    lds_barrier();
    // its elements of the QKV product (the same in every layer): row, column inside the head, rotary factors
    const SmallProd& q = m.qkv;
    const int qhalf = 1 << (q.cs - 1), qsft = q.cs - 1, qn = M << qsft;
    const int c0 = column_of<true>(q, wg, 0), which = c0 < D ? 0 : c0 < 2 * D ? 1 : 2, h = (c0 - which * D) >> 6, d0 = c0 & 63;
    float2 cs[4], sn[4];
    unsigned to[4];  // where the element goes: in the query rows, or in a layer's cache pool
    if (wg < q.units) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = min(lane + 64 * j, qn - 1), row = i >> qsft, c = (i & ((1 << qsft) - 1)) * 2;
        const int f = d0 + (c < qhalf ? c : c - qhalf), d = d0 + (c < qhalf ? c : 32 + c - qhalf), pos = sh.pos[row];
        if (which < 2) {
          cs[j] = *reinterpret_cast<const float2*>(m.rope_cos + (long)pos * 32 + f);
          sn[j] = *reinterpret_cast<const float2*>(m.rope_sin + (long)pos * 32 + f);
        }
        to[j] = which == 0 ? (unsigned)(row * D + h * 64 + d)
                           : (unsigned)((((sh.page[row] * 2 + (which - 1)) * Hh + h) * p.PT + (pos & (p.PT - 1))) * 64 + d);
      }
    }

    // ---- patch embedding ----
    const SmallProd& e = m.embed;
    if (wg < e.units) {
      if (!hop()) return;
      lds_barrier();
      bf16* x0 = v.rows(0, kIn) + (wg << e.cs);
      each_pair(e, M, lane, [&](int row, int c) {
        const float2 s = sums_of<false, false>(sh, row, c, 0, e.used).a;
        sh.xown[row][c] = s.x;
        sh.xown[row][c + 1] = s.y;
        publish_bf16x2(x0 + row * D + c, s.x, s.y);
      });
      raise();
    }
    walk.done(e.units);

    for (int l = 0; l < m.L; ++l) {
      // ---- RMSNorm + QKV + RoPE + cache write ----
      if (wg < q.units) {
        if (!hop()) return;
        bf16* dst = which == 0 ? v.rows(l, kQuery) : m.kv_pool + (size_t)l * m.layer_pool_elems;
        lds_barrier();
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int i = lane + 64 * j;
          if (64 * j >= qn) break;
          if (i < qn) {
            const int row = i >> qsft, c = (i & ((1 << qsft) - 1)) * 2;
            const Sums z = sums_of<true, true>(sh, row, c, c < qhalf ? c + qhalf : c - qhalf, q.used);
            const float rs = norm_scale(z.ss, D);
            float2 s = z.a;
            s.x *= rs;
            s.y *= rs;
            if (which < 2) {
              const float2 pv = z.b;
              const float sg = c < qhalf ? -rs : rs;
              s.x = s.x * cs[j].x + sg * pv.x * sn[j].x;
              s.y = s.y * cs[j].y + sg * pv.y * sn[j].y;
            }
            publish_bf16x2(dst + to[j], s.x, s.y);
          }
        }
        raise();
      }
      walk.done(q.units);

      // ---- attention: (series slot, head) = workgroup ----
      if (wg < n * Hh) {
        const int total = sh.pos[(wg / Hh) * nq] + nq;
        if (!hop()) return;
        attend_barriers(total);
        lds_barrier();  // (the workers have published)
        raise();
      }
      walk.done(n * Hh);

      // ---- products added to the residual: attention output, FFN down ----
      auto residual = [&](const SmallProd& d, bf16* out, bool last) -> bool {
        if (wg < d.units) {
          if (!hop()) return false;
          lds_barrier();
          const int at0 = wg << d.cs;
          float* res = v.residual();
          each_pair(d, M, lane, [&](int row, int c) {
            float2 s = sums_of<false, false>(sh, row, c, 0, d.used).a;
            s.x += sh.xown[row][c];
            s.y += sh.xown[row][c + 1];
            sh.xown[row][c] = s.x;
            sh.xown[row][c + 1] = s.y;
            const int at = row * D + at0 + c;
            if (last) {  // the head reads the fp32 residual
              publish4(res + at, __builtin_bit_cast(unsigned, s.x));
              publish4(res + at + 1, __builtin_bit_cast(unsigned, s.y));
            } else {
              publish_bf16x2(out + at, s.x, s.y);
            }
          });
          raise();
        }
        walk.done(d.units);
        return true;
      };
      if (!residual(m.out, v.rows(l, kMid), false)) return;

      // ---- RMSNorm + FFN up + GELU ----
      const SmallProd& f1 = m.up;
      if (wg < f1.units) {
        if (!hop()) return;
        lds_barrier();
        finish_up(m, v, v.rows(l, kHidden), wg, lane, sh);
        raise();
      }
      walk.done(f1.units);
      if (!residual(m.down, v.rows(l + 1, kIn), l + 1 == m.L)) return;
    }

    // ---- RMSNorm (of the fp32 residual) + head ----
    const SmallProd& hd = m.head;
    if (wg < hd.units) {
      if (!hop()) return;
      lds_barrier();
      finish_head(p, m, v, wg, lane, sh);
      raise();
    }
    walk.done(hd.units);
  }
}

// The passes of a launch: series still decoding, positions proposed, draft steps, passes.
struct Extent {
  int n, Kr, Kd, n_pass;
  __device__ __forceinline__ explicit Extent(const SmallRoundP& p) {
    n = p.counts ? min(p.counts[0], p.n) : p.n;
    Kr = p.step_only ? 0 : (p.follow_need ? max(1, min(p.K, p.counts[1])) : p.K);
    Kd = (p.phases & 1) ? Kr : 0;
    n_pass = Kd + ((p.phases & 2) ? 1 : 0);
  }
};

__global__ __launch_bounds__(kThreads) void small_round_kernel(const SmallRoundP p) {
  __shared__ __attribute__((aligned(16))) Shared sh;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Extent x(p);
  if (x.n <= 0) return;
  // (What decides here is the same for every wavefront.  The status word is not: another workgroup may set it between two looks, and
  //  wavefronts of one workgroup must not part.  Behind a launch that gave up this one may run for nothing, or leave at its first
  //  long wait; the kernel behind it goes by the word either way.)
  if (p.wait_ticks <= 0) {
    if (blockIdx.x == 0 && threadIdx.x == 0) give_up(p);
    return;
  }
  if (threadIdx.x == 0) sh.quit = 0;
  lds_barrier();
  if (wave == kWorkers)
    control_loop(p, x.n, x.Kr, x.Kd, x.n_pass, lane, sh);
  else
    worker_loop(p, x.n, x.Kr, x.Kd, x.n_pass, wave, lane, sh);
}

// The same passes from their beginning for ONE series, by a workgroup of the four workers that takes the units of a stage one after
// the other and waits for nobody: for a launch that gave up.  Nothing is lost by that: what a pass overwrites (the cache rows of
// its tokens, proposals, target means) follows from what was committed before.  Slow (some 3 us per unit and stage) and rare: from
// the next call on the handle runs kernel by kernel.  `place`: this workgroup's rows of the exchange buffer, place * nq and on.
__device__ __forceinline__ void series_alone(const SmallRoundP& p, int b, int place, Shared& sh) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Extent x(p);
  const Rsrc patches = patches_of(p);
  const int my_page = p.page_table[(long)b * p.pt_stride + min(lane, p.pt_stride - 1)];
  Weights w;
  for (int ps = 0; ps < x.n_pass; ++ps) {
    const PassView v(p, ps, x.Kd, x.Kr, 1);
    const SmallModel& m = *v.m;
    const int D = v.D, nq = v.nq, Hh = m.Hh, row0 = place * nq;
    const int base = p.len[b] + (v.draft ? (v.step == 1 ? -1 : v.step - 1) : 0);
    float* res = v.residual() + row0 * D;  // (the residual of all columns: here in memory)
    __syncthreads();
    if (threadIdx.x < kRowsMax) {
      const int pos = base + min((int)threadIdx.x, nq - 1);
      sh.ser[threadIdx.x] = b;
      sh.pos[threadIdx.x] = pos;
      sh.page[threadIdx.x] = p.page_table[(long)b * p.pt_stride + (pos >> p.pt_shift)];
    }
    __syncthreads();
    auto rows = [&](int l, int part) { return v.rows(l, part) + (long)row0 * (part == kHidden ? m.F : D); };
    // a product: the workers' share of every unit, then its epilogue
    auto units = [&](const SmallProd& d, auto share, auto finish) {
      for (int u = 0; u < d.units; ++u) {
        share(u);
        __syncthreads();
        if (wave == 0) finish(u);
        __syncthreads();
      }
    };
    auto product_of_rows = [&](const SmallProd& d, const bf16* W, const bf16* A, bool norm) {
      return [&, W, A, norm](int u) {
        prefetch<false>(d, W, u, wave, lane, w);
        product(d, A, nq, norm, wave, lane, w, sh);
      };
    };
    auto add_residual = [&](const SmallProd& d, bf16* out, bool first, bool last) {
      return [&, out, first, last](int u) {
        const int at0 = u << d.cs;
        each_pair(d, nq, lane, [&](int row, int c) {
          float2 s = sums_of<false, false>(sh, row, c, 0, d.used).a;
          float* r = res + row * D + at0 + c;
          if (!first) {
            s.x += r[0];
            s.y += r[1];
          }
          r[0] = s.x;
          r[1] = s.y;
          if (!last) publish_bf16x2(out + row * D + at0 + c, s.x, s.y);
        });
      };
    };

    units(m.embed,
          [&](int u) {
            prefetch_embed(m.embed, m.embed.W, u, wave, lane, w);
            product_f32<false>(m.embed, nq, wave, lane, w, sh, [&](int r, int k, float* f) { load_patch(p, v, sh, patches, r, k, f); });
          },
          add_residual(m.embed, rows(0, kIn), true, false));
    for (int l = 0; l < m.L; ++l) {
      bf16* pool = m.kv_pool + (size_t)l * m.layer_pool_elems;
      units(m.qkv,
            [&](int u) {
              prefetch<true>(m.qkv, v.weights(m.qkv, l), u, wave, lane, w);
              product(m.qkv, rows(l, kIn), nq, true, wave, lane, w, sh);
            },
            [&](int u) {
              const int qhalf = 1 << (m.qkv.cs - 1), c0 = column_of<true>(m.qkv, u, 0), which = c0 < D ? 0 : c0 < 2 * D ? 1 : 2;
              const int h = (c0 - which * D) >> 6, d0 = c0 & 63;
              each_pair(m.qkv, nq, lane, [&](int row, int c) {
                const int f = d0 + (c < qhalf ? c : c - qhalf), d = d0 + (c < qhalf ? c : 32 + c - qhalf), pos = sh.pos[row];
                const Sums z = sums_of<true, true>(sh, row, c, c < qhalf ? c + qhalf : c - qhalf, m.qkv.used);
                const float rs = norm_scale(z.ss, D);
                float2 s = z.a;
                s.x *= rs;
                s.y *= rs;
                if (which < 2) {
                  const float2 cs = *reinterpret_cast<const float2*>(m.rope_cos + (long)pos * 32 + f);
                  const float2 sn = *reinterpret_cast<const float2*>(m.rope_sin + (long)pos * 32 + f);
                  const float sg = c < qhalf ? -rs : rs;
                  s.x = s.x * cs.x + sg * z.b.x * sn.x;
                  s.y = s.y * cs.y + sg * z.b.y * sn.y;
                }
                bf16* to = which == 0 ? rows(l, kQuery) + (row * D + h * 64 + d)
                                      : pool + (unsigned)((((sh.page[row] * 2 + (which - 1)) * Hh + h) * p.PT + (pos & (p.PT - 1))) * 64 + d);
                publish_bf16x2(to, s.x, s.y);
              });
            });
      for (int h = 0; h < Hh; ++h) {
        attend(p, pool, rows(l, kQuery) + h * 64, rows(l, kMixed) + h * 64, D, h, Hh, my_page, base, nq, wave, lane, sh, [] { return true; });
        __syncthreads();
      }
      const bool last = l + 1 == m.L;
      units(m.out, product_of_rows(m.out, v.weights(m.out, l), rows(l, kMixed), false), add_residual(m.out, rows(l, kMid), false, false));
      units(m.up, product_of_rows(m.up, v.weights(m.up, l), rows(l, kMid), true), [&](int u) { finish_up(m, v, rows(l, kHidden), u, lane, sh); });
      units(m.down, product_of_rows(m.down, v.weights(m.down, l), rows(l, kHidden), false),
            add_residual(m.down, last ? nullptr : rows(l + 1, kIn), false, last));
    }
    units(m.head,
          [&](int u) {
            prefetch<false>(m.head, m.head.W, u, wave, lane, w);
            product_f32<true>(m.head, nq, wave, lane, w, sh, [&](int r, int k, float* f) {
              *reinterpret_cast<float4*>(f) = *reinterpret_cast<const float4*>(res + (r * D + k));
              *reinterpret_cast<float4*>(f + 4) = *reinterpret_cast<const float4*>(res + (r * D + k + 4));
            });
          },
          [&](int u) { finish_head(p, m, v, u, lane, sh); });
  }
}

// The resident launch before this kernel has finished.
__device__ __forceinline__ void mark_done(const SmallRoundP& p) {
  if (blockIdx.x == 0 && threadIdx.x == 0) __hip_atomic_store(p.done, p.done_value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Behind a launch of the resident kernel: a series per workgroup, and nothing to do (4 us) unless that launch gave up.
__global__ __launch_bounds__(kWorkers * 64) void small_round_alone_kernel(const SmallRoundP p) {
  __shared__ __attribute__((aligned(16))) Shared sh;
  if (*p.status && !(p.counts && (int)blockIdx.x >= p.counts[0])) series_alone(p, p.act ? p.act[blockIdx.x] : (int)blockIdx.x, blockIdx.x, sh);
  mark_done(p);
}

// The same at the head of the acceptance step where that follows at once: no launch of its own.
__global__ __launch_bounds__(kWorkers * 64) void small_round_accept_kernel(const SmallRoundP r, const AcceptP p) {
  __shared__ __attribute__((aligned(16))) Shared sh;
  if (*r.status && p.mode != 2) {  // (mode 2: mode 1 went before)
    const int b = p.act ? p.act[blockIdx.x] : (int)blockIdx.x;
    if (!(p.n_dev && (int)blockIdx.x >= *p.n_dev) && p.active[b]) series_alone(r, b, blockIdx.x, sh);
    __syncthreads();
  }
  mark_done(r);
  accept_step(p);
}

SmallProd product_of(const bf16* W, int K, int N) {
  const SmallPlan d = small_plan(K, N);
  return SmallProd{W, d.K, d.units, d.cs, d.per, d.used};
}

bool model_ok(const tsd_model_cfg& c, int patch) {
  const int D = c.d_model, F = c.d_ff;
  if (c.n_experts || D != 64 * c.n_heads || D > 1024 || patch > 1024) return false;
  const SmallPlan e = small_plan(patch, D);
  // (the embedding and the head, widths up to 1024, are four columns per workgroup: see product_f32)
  return small_product_ok(D, 3 * D) && small_product_ok(D, D) && small_product_ok(D, F) && small_product_ok(F, D) &&
         small_product_ok(D, patch) && e.units && e.cs == 2 && e.per <= 4 && columns_per_wg(patch) == 4;
}

}  // namespace

// The handle's decode passes can run as the resident kernel: bf16, dense, head_dim 64, at most 32 rows and 16 tokens per
// series, products that fit (and whole 16-column groups of the head: the skinny kernel's condition, whose bits these are).
bool small_round_ok(const tsd_config& c) {
  return c.dtype == TSD_BF16 && (long)c.max_batch * (c.K + 1) <= kRowsMax && c.K + 1 <= 16 && c.page_tokens >= 8 && c.patch % 16 == 0 &&
         model_ok(c.target, c.patch) && model_ok(c.draft, c.patch);
}

void small_round_model(const tsd_model_cfg& c, int patch, const bf16* W_e, const bf16* W_h, const bf16* Wqkv, const bf16* Wo, const bf16* W1,
                       const bf16* W2, SmallModel* m) {
  m->embed = product_of(W_e, patch, c.d_model);
  m->qkv = product_of(Wqkv, c.d_model, 3 * c.d_model);
  m->out = product_of(Wo, c.d_model, c.d_model);
  m->up = product_of(W1, c.d_model, c.d_ff);
  m->down = product_of(W2, c.d_ff, c.d_model);
  m->head = product_of(W_h, c.d_model, patch);
  m->L = c.n_layers;
  m->D = c.d_model;
  m->F = c.d_ff;
  m->Hh = c.n_heads;
  m->slab_bytes = small_slab_bytes(c.d_model, c.d_ff);
  m->pass_bytes = small_pass_bytes(c.n_layers, c.d_model, c.d_ff);
}

size_t small_round_exchange_bytes(const tsd_config& c) {
  return c.K * small_pass_bytes(c.draft.n_layers, c.draft.d_model, c.draft.d_ff) + small_pass_bytes(c.target.n_layers, c.target.d_model, c.target.d_ff);
}

// Most stages a launch can have (the flags' epoch advances by this much per launch).
int small_round_stages(const tsd_config& c) { return c.K * (2 + 5 * c.draft.n_layers) + 2 + 5 * c.target.n_layers; }

// ---- who else is using the device ----
// Two resident launches that no stream orders must not run together: each needs every compute unit.  And beside anything else a
// resident launch is a bad neighbour: its workgroups leave too few registers for most kernels, whose streams then take turns with it
// where launch by launch they overlap.  So a pass runs as the resident kernel only while no other handle's passes are in flight on
// another stream; with the same bits either way, nothing else depends on it.  (Two handles
// on two streams, ms for a decode of each, taking turns through an event / now: one series through 24 layers of 1024 16.8 / 14.3
// (alone 8.5), five through 8 layers of 512 5.3 / 4.4; 29 decodes of the former beside 50 of 256 series 480 / 375.)
namespace {
std::mutex uses_mutex;
std::vector<PassUse*> uses;         // of all handles
std::atomic<int> resident_handles;  // those among them that may run the resident kernel
std::atomic<long long> last_asked;  // when one of those last wanted to, in ns

// A handle's passes are numbered where others look, and its stream writes the number of the last finished one to a pinned host word: the
// kernel behind a resident launch does, behind other passes a fill kernel.  (Not events: looking at one whose stream is being
// captured by now ends that capture.)  Such a kernel per pass costs some us (an event 0.5 % of the target-only steps of 256 series), so
// other passes are marked only while somebody is asking: a small handle that starts beside busy ones takes the resident kernel until
// their next passes.
constexpr long long kAskedRecently = 100000000;
long long now_ns() { return std::chrono::duration_cast<std::chrono::nanoseconds>(std::chrono::steady_clock::now().time_since_epoch()).count(); }

std::thread::id thread_of(hipStream_t st) {  // (hipStreamPerThread names another stream in every thread)
  return st == hipStreamPerThread ? std::this_thread::get_id() : std::thread::id();
}

bool in_flight(const PassUse& u) { return u.done && __atomic_load_n(u.done, __ATOMIC_RELAXED) != u.launched; }

// The number of the pass now launched on `st`.
int number_pass(PassUse* use, hipStream_t st) {
  use->stream = st;
  use->thread = thread_of(st);
  return ++use->launched;
}
}  // namespace

void add_use(PassUse* use, int device, bool resident, int* done) {
  std::lock_guard<std::mutex> lock(uses_mutex);
  use->device = device;
  use->resident = resident;
  use->done = done;
  uses.push_back(use);
  if (resident) ++resident_handles;
}

void remove_use(PassUse* use) {
  std::lock_guard<std::mutex> lock(uses_mutex);
  uses.erase(std::remove(uses.begin(), uses.end(), use), uses.end());
  if (use->resident) --resident_handles;
}

hipError_t note_pass(PassUse* use, hipStream_t st) {
  if (resident_handles.load(std::memory_order_relaxed) <= (use->resident ? 1 : 0) || !use->done) return hipSuccess;  // nobody else could ask,
  if (now_ns() - last_asked.load(std::memory_order_relaxed) > kAskedRecently) return hipSuccess;                    // or does
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (st) {
    hipError_t e = hipStreamIsCapturing(st, &cs);
    if (e != hipSuccess || cs != hipStreamCaptureStatusNone) return e;
  }
  std::lock_guard<std::mutex> lock(uses_mutex);
  return launch_fill_int(use->done, number_pass(use, st), 1, st);
}

hipError_t launch_small_round(SmallRoundP& p, PassUse* use, hipStream_t st, bool* busy) {
  *busy = false;
  last_asked.store(now_ns(), std::memory_order_relaxed);
  std::lock_guard<std::mutex> lock(uses_mutex);
  for (const PassUse* u : uses)
    if (u != use && u->device == use->device && in_flight(*u) && (u->stream != st || u->thread != thread_of(st))) {
      *busy = true;
      return hipSuccess;
    }
  p.done = use->done;
  p.done_value = number_pass(use, st);
  hipLaunchKernelGGL(small_round_kernel, dim3(kWg), dim3(kThreads), 0, st, p);
  return hipGetLastError();
}

hipError_t launch_small_round_alone(const SmallRoundP& p, hipStream_t st) {
  hipLaunchKernelGGL(small_round_alone_kernel, dim3(p.n), dim3(kWorkers * 64), 0, st, p);
  return hipGetLastError();
}

hipError_t launch_small_round_accept(const SmallRoundP& r, const AcceptP& p, hipStream_t st) {
  hipLaunchKernelGGL(small_round_accept_kernel, dim3(p.B), dim3(kWorkers * 64), 0, st, r, p);
  return hipGetLastError();
}

}  // namespace tsd
