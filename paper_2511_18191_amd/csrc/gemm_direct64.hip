// Small-tile bf16 GEMM for products that leave at most one 64 x 64 tile per compute unit, or two: C[M,N] = A[M,K] * Wt[N,K]^T
// with the fused epilogues of the tiled family (gemm_epilogue.h).  Both operands go from global memory straight into LDS
// (global_load_lds_dwordx4: no staging registers, no LDS writes by the lanes) through a ring of four stages of one 64-wide
// k-tile each.  (Larger products: gemm_wide.hip.)
//
// Four wavefronts of 32 x 32 leave a k-tile only 4 MFMAs per wavefront, so what bounds such a tile is the way of its
// operands from L2 or HBM; four k-tiles in flight (64 KB, two workgroups per compute unit) are the best ring: 1280x512x512
// 5.0 us, 558x1536x512 6.1, 256x2048x512 5.2.  Of the other depths three (48 KB, three workgroups) is as fast alone and
// 2 % slower in a whole pass of 93 series, where the weights come from HBM; six (one workgroup) is 10 % slower.
//
//   * A stage is its rows back to back (A rows, then B rows), 128 bytes per row; the eight 16-byte chunks of a row
//     sit at chunk ^ ((row >> 1) & 7), which makes the fragment reads (32 consecutive rows, one chunk; or 16 and two) conflict-free
//     without padding.  A load instruction fills 1 KB = 8 rows; lane l fetches the chunk that belongs at l.
//   * A wavefront owns one contiguous run of every stage and addresses its loads through the instruction's immediate
//     offset around one base, so M0 (the LDS base of such a load) is written once per k-tile.
//   * The fragments of a k-tile are requested from LDS a k-tile ahead.  One barrier per k-tile: by then every wavefront holds all of the
//     k-tile's fragments in registers, so the k-tile's own slot is refilled at once.
//   * The RMSNorm row sums come from the A fragments on their way to the matrix cores (A never sits in registers
//     otherwise), in the summation order of the register-staged kernel (gemm.hip): per row eight partial sums, one per
//     16-byte chunk position of a 64-wide k-run, each a chain of packed bf16 dot products, combined as
//     ((P0 + P4) + (P2 + P6)) + ((P1 + P5) + (P3 + P7)).  The products accumulate k in the same order with the
//     same instruction, so all kernels give the same bits and the launcher may pick any by the product's shape.
//     (Contexts of small handles have the sums of gemm_skinny.hip instead: kShares.)
#include "direct_lds.h"
#include "gemm_epilogue.h"
#include "tile_order.h"

namespace tsd {

namespace d64 {

constexpr int BM = 64, BN = 64, BK = 64, NS = 4;  // tile, stages
constexpr int NW = 4, NT = NW * 64;               // wavefronts, 2 x 2 blocks of 32 x 32
constexpr int ROWB = BK * 2, CPR = ROWB / 16;     // bytes and 16-byte chunks of a stage row
constexpr int RPL = 1024 / ROWB;                  // rows a load instruction covers
constexpr int STAGE = (BM + BN) * ROWB;
constexpr int NL = STAGE / 1024 / NW;             // load instructions of a wavefront per stage
constexpr int REGION = NL * 1024;                 // a wavefront's bytes of a stage
constexpr int BIAS = REGION / 2;                  // M0 points here inside the region: immediates stay small
constexpr int LDC = BN + 4;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr int kSc1 = 16;  // cache policy of what workgroups hand each other: agent scope
constexpr size_t SMEM = (size_t)NS * STAGE + BM * 12;  // stages, then row_scale / row_pos / row_page
static_assert(64 * LDC * 4 <= NS * STAGE, "the epilogue's buffer reuses the stages");

// (v[l] + v[l ^ 16]) + (v[l ^ 32] + v[l ^ 48]), lanes exchanged in registers
__device__ __forceinline__ float add_quarters(float v) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  const unsigned half = __float_as_uint(__uint_as_float(p[0]) + __uint_as_float(p[1]));
  const auto q = __builtin_amdgcn_permlane32_swap(half, half, false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// How a tile sums over k.
enum Sums {
  kWhole,   // in one run, long contractions of activations in four (see gemm.hip)
  kOneRun,  // (EP_STORE) p.K is one run of a longer contraction, its sums are for another workgroup of the launch
  // As gemm_skinny.hip: a share per wavefront of its workgroups, 32 k at a time, the shares added in order (same bits).  What it costs over
  // kWhole is the vector arithmetic at a share's end, every 32 k at K = 512, and the chains of row sums (145x1536x512 7.6 us against
  // 5.8, without the norm 145x512x512 5.5 against 5.1); the MFMAs of a first step without an addend gained nothing (7.5).
  kShares,
};

// Rows m0 .. min(m0 + 64, M) - 1, columns n0 .. n0 + 63, by a workgroup of NT lanes.  ldk: elements between rows of A and of W.
template <int AM, int EP, Sums SUMS>
__device__ __forceinline__ void tile64(const GemmP& p, int ldk, int M, int m0, int n0, unsigned char* smem) {
  constexpr bool kNorm = (AM == A_NORM), kSkinny = SUMS == kShares;
  float* Cs = reinterpret_cast<float*>(smem);                            // [64][LDC], after the main loop
  float* row_scale = reinterpret_cast<float*>(smem + NS * STAGE);        // [BM]
  int* row_pos = reinterpret_cast<int*>(smem + NS * STAGE + BM * 4);     // [BM] EP_QKV
  int* row_page = row_pos + BM;                                          // [BM] EP_QKV
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wid >> 1, wn = wid & 1;
  const int N = p.N, K = p.K;

  // Epilogue inputs that do not depend on the product are requested before the operands (loads return in order, so nothing
  // older than the stages' loads disturbs their counted waits) and land behind the main loop.
  int2 my_meta = make_int2(0, 0);
  if constexpr (EP == EP_QKV) {
    my_meta = p.row_meta[min(m0 + min(tid, BM - 1), M - 1)];
  }

  constexpr int NPRE = (EP == EP_RESID) ? 64 * (BN / 4) / NT : 1;
  float4 oldc[NPRE];
  if constexpr (EP == EP_RESID) {
#pragma unroll
    for (int it = 0; it < NPRE; ++it) {
      const int g = tid + it * NT;
      const int gm = min(m0 + g / (BN / 4), M - 1), gn = n0 + (g % (BN / 4)) * 4;  // (N is a multiple of BN)
      oldc[it] = *reinterpret_cast<const float4*>(p.Cf + (long)gm * N + gn);
    }
  }

  // ---- loads: wavefront w fills the stage rows [NL * RPL * w, NL * RPL * (w + 1)); stage row R is A row R (R < BM) or B
  // row R - BM.  Lane l of load j covers row (w NL + j) RPL + l / CPR and the physical chunk l % CPR of it, i.e. the
  // logical chunk (l % CPR) ^ swizzle(row).  The immediate of load j (j * 1024 - BIAS) is added to BOTH addresses by the
  // instruction, so it is taken off the global pointer here.
  auto swizzle = [](int R) { return (R >> 1) & 7; };
  const bf16* Ap = reinterpret_cast<const bf16*>(p.A);
  const bf16* Wp = reinterpret_cast<const bf16*>(p.W);
  const bf16* gp[NL];
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const int R = (wid * NL + j) * RPL + lane / CPR;
    const int chunk = (lane % CPR) ^ swizzle(R);
    const bf16* row;
    if ((wid * NL + j) * RPL < BM) {  // (uniform per instruction: BM is a multiple of the rows it covers)
      row = Ap + (long)min(m0 + R, M - 1) * ldk;  // rows past M are clamped to the last row: their products are never stored
    } else {
      row = Wp + (long)(n0 + R - BM) * ldk;
    }
    gp[j] = row + chunk * 8 - (j * 1024 - BIAS) / 2;
  }
  auto issue_stage = [&](int slot, int kt) {
    issue_loads<0, NL, BIAS>(gp, (long)kt * BK, TSD_LDS_PTR(smem + slot * STAGE + wid * REGION + BIAS));
  };

  // ---- fragments: lane l reads row l % 32 of a 32-row block, chunk 2 s + l / 32 of k16 sub-step s (kShares: row l % 16 of 16-row block s % 2,
  // chunk 4 (s / 2) + l / 16 of k32 step s / 2)
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  // Long contractions of activations are summed in four runs of ceil(nk / 4) k-tiles, each from zero, the runs added in
  // order (the order of the split workgroups of gemm.hip, which every kernel that can take such a product keeps to)
  constexpr bool kQuarters = AM == A_ACT && SUMS == kWhole;
  f32x16 tot;
  float ss[4] = {0.f, 0.f, 0.f, 0.f};  // row-sum chains of this lane: chunk positions hi, 2 + hi, 4 + hi, 6 + hi of a 64-wide k-run
  const int r31 = lane & 31, hi = lane >> 5, l15 = lane & 15, lg = lane >> 4;
  const int RA = wm * 32 + (kSkinny ? l15 : r31), RB = BM + wn * 32 + (kSkinny ? l15 : r31);
  // kShares: the share's sums, the shares' sums so far; k32 steps of a share, and those still to come of the one under way
  f32x4 part[2][2], sum[2][2];
#pragma unroll
  for (int i = 0; i < 4; ++i) part[i >> 1][i & 1] = sum[i >> 1][i & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
  float share_ss = 0.f, sum_ss = 0.f;  // row sums of this wavefront's 16-row block number wn
  const int share = (K / 32 + skinny_shares(K) - 1) / skinny_shares(K);
  int left = share;
  auto end_share = [&] {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        sum[i][j] += part[i][j];
        part[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    if constexpr (kNorm) {
      sum_ss += add_quarters(share_ss);
      share_ss = 0.f;
    }
    left = share;
  };
  const int offA = RA * ROWB, offB = RB * ROWB, swA = swizzle(RA), swB = swizzle(RB);

  // The k loop: a k-tile is four k16 sub-steps, one MFMA each, a chain of dependent sums that leaves LDS latency nothing to hide behind.
  // So the fragments of a whole k-tile are requested at once, a k-tile ahead, in two sets in turn (with one sub-step of lookahead
  // 256x1536x512 took 5.96 us instead of 5.80, 256x2304x768 7.03 / 6.80, 256x3072x1024 8.13 / 7.75).  One barrier per k-tile:
  //   this wavefront's loads of k-tile kt + 1 are done (only those of later k-tiles may still be in flight) and its
  //   fragments of k-tile kt all sit in registers (LDS counter at zero);
  //   after the barrier that holds for everybody, so k-tile kt + 1 can be read and the slot of k-tile kt itself refilled
  //   with k-tile kt + NS.
  // (a bare s_barrier: __syncthreads() would also wait for every load in flight)
  bf16x8 fa[2][4], fb[2][4];
  auto read_frags = [&](auto set, int kt) {
    constexpr int F = decltype(set)::value;
    const unsigned char* st = smem + (kt % NS) * STAGE;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      // (rows 16 apart have the same swizzle)
      const int chunk = kSkinny ? 4 * (s >> 1) + lg : 2 * s + hi, block = kSkinny ? (s & 1) * 16 * ROWB : 0;
      fa[F][s] = *reinterpret_cast<const bf16x8*>(st + offA + block + ((chunk ^ swA) << 4));
      fb[F][s] = *reinterpret_cast<const bf16x8*>(st + offB + block + ((chunk ^ swB) << 4));
    }
  };
  // One k-tile.  SET: its fragments; PEND: the loads this wavefront may leave in flight at the barrier (those of the k-tiles after
  // kt + 1), or -1 for the last k-tile (no barrier, nothing left to read); REFILL: k-tile kt + NS exists.
  auto tile = [&](auto set, int kt, auto pend, auto refill) {
    constexpr int F = decltype(set)::value, PEND = decltype(pend)::value;
    constexpr bool REFILL = decltype(refill)::value != 0;
    if constexpr (PEND >= 0) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(PEND) : "memory");
#pragma unroll
    for (int s = 0; s < 4; ++s) asm volatile("" : "+v"(fa[F][s]), "+v"(fb[F][s]));  // (waited for here, not behind the next set's requests)
    if constexpr (PEND >= 0) read_frags(IC<1 - F>{}, kt + 1);
    if constexpr (REFILL) issue_stage(kt % NS, kt + NS);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kSkinny) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) part[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[F][2 * t + i], fb[F][2 * t + j], part[i][j], 0, 0, 0);
        if constexpr (kNorm) {
          const bf16x8 a = wn ? fa[F][2 * t + 1] : fa[F][2 * t];
#pragma unroll
          for (int e = 0; e < 8; ++e) share_ss = fmaf((float)a[e], (float)a[e], share_ss);
        }
        if (--left == 0) end_share();
      }
      __builtin_amdgcn_sched_barrier(0);
      return;
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if constexpr (kNorm) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bf16x2 pr = {fa[F][s][2 * e], fa[F][s][2 * e + 1]};
          ss[s] = __builtin_amdgcn_fdot2_f32_bf16(pr, pr, ss[s], false);
        }
      }
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[F][s], fb[F][s], acc, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- main loop (K is a multiple of 64, at least NS of them) ------------------------------------------------------
  const int nk = K / BK;
#pragma unroll
  for (int s = 0; s < NS; ++s) issue_stage(s, s);
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 1) * NL) : "memory");  // k-tile 0 has landed for everybody
  // steady state: k-tiles 0 .. nk - NS - 1 (each refills its slot); then the last NS k-tiles, the first of them with set 0
  const int n_steady = nk - NS;
  const bool quarters = kQuarters && K >= kQuarterK;
  const int run = (nk + 3) / 4;
  auto fold = [&](int done) {  // `done` k-tiles are in acc: at a run's end move them into the running sum
    if constexpr (kQuarters) {
      if (!quarters || done % run != 0 || done >= nk) return;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        tot[r] = done == run ? acc[r] : tot[r] + acc[r];
        acc[r] = 0.f;
      }
    }
  };
  int kt = 0;
  auto steady = [&](auto set) {
    tile(set, kt, IC<(NS - 2) * NL>{}, IC<1>{});
    fold(++kt);
  };
  if (n_steady & 1) {
    read_frags(IC<1>{}, 0);
    steady(IC<1>{});
  } else {
    read_frags(IC<0>{}, 0);
  }
  while (kt < n_steady) {
    steady(IC<0>{});
    steady(IC<1>{});
  }
  // tail: k-tile nk - NS + t leaves NS - 2 - t stages in flight at its barrier; the last one has no barrier
  auto tail = [&](auto self, auto tc) {
    constexpr int t = decltype(tc)::value;
    if constexpr (t + 1 < NS) {
      tile(IC<t & 1>{}, kt + t, IC<(NS - 2 - t) * NL>{}, IC<0>{});
      fold(kt + t + 1);
      self(self, IC<t + 1>{});
    } else {
      tile(IC<t & 1>{}, kt + t, IC<-1>{}, IC<0>{});
    }
  };
  tail(tail, IC<0>{});
  if constexpr (kQuarters) {
    if (quarters) {  // the last run joins the sum of the first three
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = tot[r] + acc[r];
    }
  }

  if constexpr (kSkinny) {
    if (left != share) end_share();
  }

  if constexpr (EP == EP_QKV) {
    if (tid < BM) {
      row_pos[tid] = my_meta.x;
      row_page[tid] = my_meta.y;
    }
  }
  // ---- RMSNorm row scale: this lane's chains are the chunk positions hi, 2 + hi, 4 + hi, 6 + hi ---------------------------
  if constexpr (kNorm && kSkinny) {
    if (lg == 0) row_scale[wm * 32 + wn * 16 + l15] = rsqrtf(sum_ss / (float)K + kRmsEps);
  } else if constexpr (kNorm) {
    const float b = (ss[0] + ss[2]) + (ss[1] + ss[3]);  // (P[hi] + P[4 + hi]) + (P[2 + hi] + P[6 + hi])
    const float all = b + __shfl_xor(b, 32);
    if (wn == 0 && hi == 0) row_scale[RA] = rsqrtf(all / (float)K + kRmsEps);
  }

  // ---- epilogue through LDS ---------------------------------------------------------------------------------------
  auto read_c4 = [&](int row, int col) { return *reinterpret_cast<const float4*>(Cs + row * LDC + col); };
  __syncthreads();  // the stages are no longer read
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if constexpr (kSkinny) Cs[(wm * 32 + (r >> 3) * 16 + lg * 4 + (r & 3)) * LDC + wn * 32 + (r >> 2 & 1) * 16 + l15] = sum[r >> 3][r >> 2 & 1][r & 3];
    else Cs[(wm * 32 + (r >> 2) * 8 + hi * 4 + (r & 3)) * LDC + wn * 32 + r31] = acc[r];
  }
  __syncthreads();
  if constexpr (SUMS == kOneRun) {  // written through to memory
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(p.Cf, 0, 0x7fffffff, 0x00020000);
#pragma unroll
    for (int it = 0; it < 64 * (BN / 4) / NT; ++it) {
      const int g = tid + it * NT, row = g / (BN / 4), col = g % (BN / 4) * 4;
      if (m0 + row < M)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, read_c4(row, col)), rsrc, (int)(((long)(m0 + row) * N + n0 + col) * 4), 0, kSc1);
    }
  } else {
    epilogue_pass<bf16, EP, kNorm, BN, NT, EP == EP_RESID>(p, read_c4, row_scale, row_pos, row_page, m0, n0, 0, M, N, tid, oldc);
  }
}

// x += A W^T for rows m0 .. min(m0 + 64, M) - 1, columns n0 .. n0 + 63, one of the four runs of the contraction (K >= kQuarterK: see gemm.hip) per
// workgroup: each stores its 64 x 64 sums to `parts` (part_elems apart), the last one to finish, by the tile's counter, adds the four in
// order and leaves the counter at zero.  Nothing waits for another workgroup.  What the other three wrote has gone through to memory
// before they counted, and nobody has read those lines in this launch, so the loads past L1 find it.
// word: of LDS, behind the tile's.  Cb may not be NULL.
__device__ __forceinline__ void resid_run64(const bf16* A, const bf16* W, int K, float* x, bf16* xb, int N, float* parts, long part_elems, int run,
                                            unsigned* count, int M, int m0, int n0, unsigned char* smem, int* word) {
  const int tid = threadIdx.x, nk = K >> 6, r = (nk + 3) >> 2;
  GemmP g;
  g.N = N;
  g.K = min(r, nk - run * r) * 64;
  g.A = A + run * r * 64;
  g.W = W + run * r * 64;
  g.Cf = parts + run * part_elems;
  g.Cb = nullptr;
  tile64<A_ACT, EP_STORE, kOneRun>(g, K, M, m0, n0, smem);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // every wavefront's sums are there
  __syncthreads();
  if (tid == 0) *word = (int)__hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (*word != 3) return;
  if (tid == 0) __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  constexpr int NI = BM * (BN / 4) / NT;
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(parts, 0, 0x7fffffff, 0x00020000);
  float4 v[NI][4], old[NI];
  auto at = [&](int i) { return (long)min(m0 + (tid >> 4) + 16 * i, M - 1) * N + n0 + (tid & 15) * 4; };
#pragma unroll
  for (int i = 0; i < NI; ++i) {
#pragma unroll
    for (int w = 0; w < 4; ++w) v[i][w] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)((w * part_elems + at(i)) * 4), 0, kSc1));
    old[i] = *reinterpret_cast<const float4*>(x + at(i));
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    float4 s = v[i][0];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      s.x += v[i][w].x;
      s.y += v[i][w].y;
      s.z += v[i][w].z;
      s.w += v[i][w].w;
    }
    s.x = old[i].x + s.x;
    s.y = old[i].y + s.y;
    s.z = old[i].z + s.z;
    s.w = old[i].w + s.w;
    if (m0 + (tid >> 4) + 16 * i < M) {
      *reinterpret_cast<float4*>(x + at(i)) = s;
      store4<bf16>(xb + at(i), s);
    }
  }
}

}  // namespace d64

template <int AM, int EP, d64::Sums SUMS>
__global__ __launch_bounds__(d64::NT, 2) void gemm_direct64_kernel(const GemmP p) {
  using namespace d64;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  // rows of the product: fixed at launch, or capped by a device-side series count (workgroups past the cap leave)
  const int M = p.n_dev ? min(p.M, *p.n_dev * p.nq) : p.M;
  int tm, tn;
  if (!own_tile((M + BM - 1) / BM, p.N / BN, tm, tn)) return;
  const int m0 = tm * BM, n0 = tn * BN;
  tile64<AM, EP, SUMS>(p, p.K, M, m0, n0, smem);
}

// The long contractions of few rows, x += A W^T, a run of the four per workgroup (resid_run64).  With one workgroup per tile, whatever its
// wavefronts do, the few busy compute units pull 0.5 to 0.8 MB of operands each at 75 GB/s; here four times as many share them (figures
// of both at takes_runs; inside target-only steps of 256 series 256x512x2048 takes 10.3 us split, 7.8 here).
__global__ __launch_bounds__(d64::NT, 2) void gemm_runs_kernel(const GemmP p) {
  using namespace d64;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int M = p.n_dev ? min(p.M, *p.n_dev * p.nq) : p.M;
  const int tiles_m = (M + BM - 1) / BM, n_tasks = tiles_m * (p.N / BN) * 4;
  // every XCD takes one contiguous run of the tasks, the four runs of a tile next to each other, row tiles of one column next
  const int per_xcd = ((n_tasks >> 2) + 7) / 8 * 4;
  if ((int)(blockIdx.x >> 3) >= per_xcd) return;
  const int lin = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (lin >= n_tasks) return;
  const int tile = lin >> 2, tn = tile / tiles_m, tm = tile - tn * tiles_m;
  resid_run64(reinterpret_cast<const bf16*>(p.A), reinterpret_cast<const bf16*>(p.W), p.K, p.Cf, reinterpret_cast<bf16*>(p.Cb), p.N, p.parts,
              (long)kRunTiles * BM * BN, lin & 3, p.counts + tile, M, tm * BM, tn * BN, smem, reinterpret_cast<int*>(smem + SMEM));
}

// ---- host side -------------------------------------------------------------------------------------------------
template <int AM, int EP, d64::Sums SUMS = d64::kWhole>
static hipError_t launch_t(const GemmP& p, hipStream_t st) {
  const long tiles = (long)((p.M + d64::BM - 1) / d64::BM) * (p.N / d64::BN);
  hipLaunchKernelGGL((gemm_direct64_kernel<AM, EP, SUMS>), dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(d64::NT), d64::SMEM, st, p);
  return hipGetLastError();
}

hipError_t launch_gemm_direct64(int amode, int epi, const GemmP& p, hipStream_t st) {
  if (amode == A_ACT && epi == EP_STORE) return launch_t<A_ACT, EP_STORE>(p, st);
  if (amode == A_ACT && epi == EP_RESID) return launch_t<A_ACT, EP_RESID>(p, st);
  if (amode == A_NORM && epi == EP_STORE) return launch_t<A_NORM, EP_STORE>(p, st);
  if (amode == A_NORM && epi == EP_GELU) return launch_t<A_NORM, EP_GELU>(p, st);
  if (amode == A_NORM && epi == EP_QKV) return launch_t<A_NORM, EP_QKV>(p, st);
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_shares(int amode, int epi, const GemmP& p, hipStream_t st) {
  if (amode == A_ACT && epi == EP_RESID) return launch_t<A_ACT, EP_RESID, d64::kShares>(p, st);
  if (amode == A_NORM && epi == EP_GELU) return launch_t<A_NORM, EP_GELU, d64::kShares>(p, st);
  if (amode == A_NORM && epi == EP_QKV) return launch_t<A_NORM, EP_QKV, d64::kShares>(p, st);
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_runs(const GemmP& p, hipStream_t st) {
  const long tiles = (long)((p.M + d64::BM - 1) / d64::BM) * (p.N / d64::BN);
  hipLaunchKernelGGL(gemm_runs_kernel, dim3((unsigned)((tiles + 7) / 8 * 32)), dim3(d64::NT), d64::SMEM + 64, st, p);
  return hipGetLastError();
}

template <int AM, int EP, d64::Sums SUMS = d64::kWhole>
static hipError_t raise() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_direct64_kernel<AM, EP, SUMS>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)d64::SMEM);
}

// More than 64 KB of dynamic LDS needs a one-time opt-in per kernel, outside any stream capture.
hipError_t prepare_gemm_direct64() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_runs_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)d64::SMEM + 64);
  if (e != hipSuccess) return e;
  if ((e = raise<A_ACT, EP_STORE>()) != hipSuccess) return e;
  if ((e = raise<A_ACT, EP_RESID>()) != hipSuccess) return e;
  if ((e = raise<A_NORM, EP_STORE>()) != hipSuccess) return e;
  if ((e = raise<A_NORM, EP_GELU>()) != hipSuccess) return e;
  if ((e = raise<A_NORM, EP_QKV>()) != hipSuccess) return e;
  if ((e = raise<A_ACT, EP_RESID, d64::kShares>()) != hipSuccess) return e;
  if ((e = raise<A_NORM, EP_GELU, d64::kShares>()) != hipSuccess) return e;
  return raise<A_NORM, EP_QKV, d64::kShares>();
}

}  // namespace tsd
