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
//     sit at chunk ^ ((row >> 1) & 7), which makes the fragment reads (32 consecutive rows, one chunk) conflict-free
//     without padding.  A load instruction fills 1 KB = 8 rows; lane l fetches the chunk that belongs at l.
//   * A wavefront owns one contiguous run of every stage and addresses its loads through the instruction's immediate
//     offset around one base, so M0 (the LDS base of such a load) is written once per k-tile.
//   * The k loop is software-pipelined by k16 sub-steps: while the MFMAs of one sub-step run, the fragments of the next
//     are on their way from LDS, also across k-tiles.  One barrier per k-tile, before its LAST sub-step: by then every
//     wavefront holds all of the k-tile's fragments in registers, so the k-tile's own slot is refilled at once.
//   * The RMSNorm row sums come from the A fragments on their way to the matrix cores (A never sits in registers
//     otherwise), in the summation order of the register-staged kernel (gemm.hip): per row eight partial sums, one per
//     16-byte chunk position of a 64-wide k-run, each a chain of packed bf16 dot products, combined as
//     ((P0 + P4) + (P2 + P6)) + ((P1 + P5) + (P3 + P7)).  The products accumulate k in the same order with the
//     same instruction, so all kernels give the same bits and the launcher may pick any by the product's shape.
#include "direct_lds.h"
#include "gemm_epilogue.h"

namespace tsd {

namespace {
constexpr int BM = 64, BN = 64, BK = 64, NS = 4;  // tile, stages
constexpr int NW = 4, NT = NW * 64;               // wavefronts, 2 x 2 blocks of 32 x 32
constexpr int ROWB = BK * 2, CPR = ROWB / 16;     // bytes and 16-byte chunks of a stage row
constexpr int RPL = 1024 / ROWB;                  // rows a load instruction covers
constexpr int STAGE = (BM + BN) * ROWB;
constexpr int NL = STAGE / 1024 / NW;             // load instructions of a wavefront per stage
constexpr int REGION = NL * 1024;                 // a wavefront's bytes of a stage
constexpr int BIAS = REGION / 2;                  // M0 points here inside the region: immediates stay small
constexpr int LDC = BN + 4;
constexpr size_t SMEM = (size_t)NS * STAGE + BM * 12;  // stages, then row_scale / row_pos / row_page
static_assert(64 * LDC * 4 <= NS * STAGE, "the epilogue's buffer reuses the stages");
}  // namespace

template <int AM, int EP>
__global__ __launch_bounds__(NT, 2) void gemm_direct64_kernel(const GemmP p) {
  constexpr bool kNorm = (AM == A_NORM);
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  float* Cs = reinterpret_cast<float*>(smem);                            // [64][LDC], after the main loop
  float* row_scale = reinterpret_cast<float*>(smem + NS * STAGE);        // [BM]
  int* row_pos = reinterpret_cast<int*>(smem + NS * STAGE + BM * 4);     // [BM] EP_QKV
  int* row_page = row_pos + BM;                                          // [BM] EP_QKV

  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wid >> 1, wn = wid & 1;
  // rows of the product: fixed at launch, or capped by a device-side series count (workgroups past the cap leave)
  const int M = p.n_dev ? min(p.M, *p.n_dev * p.nq) : p.M;
  const int N = p.N, K = p.K;
  // tile order: every XCD walks one contiguous run of the tile list, the list ordered in groups of 8 tile columns
  // walked row by row (see gemm.hip)
  const int tiles_m = (M + BM - 1) / BM, tiles_n = N / BN;
  const int n_tiles = tiles_m * tiles_n;
  const int per_xcd = (n_tiles + 7) >> 3;
  if ((int)(blockIdx.x >> 3) >= per_xcd) return;
  const int lin = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (lin >= n_tiles) return;
  constexpr int GW = 8;
  const int gc = lin / (GW * tiles_m), rem = lin - gc * (GW * tiles_m);
  const int gw = min(GW, tiles_n - gc * GW);
  const int tm = rem / gw, tn = gc * GW + rem - tm * gw;
  const int m0 = tm * BM, n0 = tn * BN;

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
      row = Ap + (long)min(m0 + R, M - 1) * K;  // rows past M are clamped to the last row: their products are never stored
    } else {
      row = Wp + (long)(n0 + R - BM) * K;
    }
    gp[j] = row + chunk * 8 - (j * 1024 - BIAS) / 2;
  }
  auto issue_stage = [&](int slot, int kt) {
    issue_loads<0, NL, BIAS>(gp, (long)kt * BK, TSD_LDS_PTR(smem + slot * STAGE + wid * REGION + BIAS));
  };

  // ---- fragments: lane l reads row l % 32 of a 32-row block, chunk 2 s + l / 32 of k16 sub-step s
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  // Long contractions of activations are summed in four runs of ceil(nk / 4) k-tiles, each from zero, the runs added in
  // order (the order of the split workgroups of gemm.hip, which every kernel that can take such a product keeps to)
  constexpr bool kQuarters = AM == A_ACT;
  f32x16 tot;
  float ss[4] = {0.f, 0.f, 0.f, 0.f};  // row-sum chains of this lane: chunk positions hi, 2 + hi, 4 + hi, 6 + hi of a 64-wide k-run
  const int r31 = lane & 31, hi = lane >> 5;
  const int RA = wm * 32 + r31, RB = BM + wn * 32 + r31;
  const int offA = RA * ROWB, offB = RB * ROWB, swA = swizzle(RA), swB = swizzle(RB);

  // The k loop by k16 sub-steps (two fragment reads, one MFMA each), two fragment sets F[0], F[1] in turn:
  //   sub-step s of k-tile kt:   read F[(s + 1) & 1] <- the next sub-step;   MFMAs on F[s & 1]
  // and before the read of the LAST sub-step's successor (sub-step 0 of k-tile kt + 1) the barrier of k-tile kt:
  //   this wavefront's loads of k-tile kt + 1 are done (only those of later k-tiles may still be in flight) and its
  //   fragments of k-tile kt all sit in registers (LDS counter at zero: they were requested a sub-step's MFMAs ago);
  //   after the barrier that holds for everybody, so k-tile kt + 1 can be read and the slot of k-tile kt itself refilled
  //   with k-tile kt + NS.
  // (a bare s_barrier: __syncthreads() would also wait for every load in flight)
  bf16x8 fa[2], fb[2];
  auto read_frags = [&](int kt, int s) {
    const unsigned char* st = smem + (kt % NS) * STAGE;
    fa[s & 1] = *reinterpret_cast<const bf16x8*>(st + offA + (((2 * s + hi) ^ swA) << 4));
    fb[s & 1] = *reinterpret_cast<const bf16x8*>(st + offB + (((2 * s + hi) ^ swB) << 4));
  };
  // `arrived`: an empty statement that uses a fragment set, placed BEFORE the next set's reads are issued.  The compiler
  // waits for LDS data right before its first use and cannot tell the two sets' reads apart by count here, so without it
  // the wait would land after the next set's reads were issued and cover those too (a full LDS round trip exposed per
  // sub-step); with it the wait covers only reads issued a sub-step ago, which have long landed.
  // One k-tile.  PEND: the loads this wavefront may leave in flight at the barrier (those of the k-tiles after kt + 1), or
  // -1 for the last k-tile (no barrier, nothing left to read); REFILL: k-tile kt + NS exists.
  auto tile = [&](int kt, auto pend, auto refill) {
    constexpr int PEND = decltype(pend)::value;
    constexpr bool REFILL = decltype(refill)::value != 0;
    const auto sub = [&](auto sc) {
      constexpr int s = decltype(sc)::value;
      asm volatile("" : "+v"(fa[s & 1]), "+v"(fb[s & 1]));
      if constexpr (s < 3) {
        read_frags(kt, s + 1);
      } else if constexpr (PEND >= 0) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(PEND) : "memory");
        if constexpr (REFILL) issue_stage(kt % NS, kt + NS);
        read_frags(kt + 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (kNorm) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bf16x2 pr = {fa[s & 1][2 * e], fa[s & 1][2 * e + 1]};
          ss[s] = __builtin_amdgcn_fdot2_f32_bf16(pr, pr, ss[s], false);
        }
      }
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s & 1], fb[s & 1], acc, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    sub(IC<0>{});
    sub(IC<1>{});
    sub(IC<2>{});
    sub(IC<3>{});
  };

  // ---- main loop (K is a multiple of 64, at least NS of them) ------------------------------------------------------
  const int nk = K / BK;
#pragma unroll
  for (int s = 0; s < NS; ++s) issue_stage(s, s);
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 1) * NL) : "memory");  // k-tile 0 has landed for everybody
  read_frags(0, 0);
  // steady state: k-tiles 0 .. nk - NS - 1 (each refills its slot); then the last NS k-tiles
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
  for (; kt < n_steady; ++kt) {
    tile(kt, IC<(NS - 2) * NL>{}, IC<1>{});
    fold(kt + 1);
  }
  // tail: k-tile nk - NS + t leaves NS - 2 - t stages in flight at its barrier; the last one has no barrier
  auto tail = [&](auto self, auto tc) {
    constexpr int t = decltype(tc)::value;
    if constexpr (t + 1 < NS) {
      tile(kt + t, IC<(NS - 2 - t) * NL>{}, IC<0>{});
      fold(kt + t + 1);
      self(self, IC<t + 1>{});
    } else {
      tile(kt + t, IC<-1>{}, IC<0>{});
    }
  };
  tail(tail, IC<0>{});
  if constexpr (kQuarters) {
    if (quarters) {  // the last run joins the sum of the first three
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = tot[r] + acc[r];
    }
  }

  if constexpr (EP == EP_QKV) {
    if (tid < BM) {
      row_pos[tid] = my_meta.x;
      row_page[tid] = my_meta.y;
    }
  }
  // ---- RMSNorm row scale: this lane's chains are the chunk positions hi, 2 + hi, 4 + hi, 6 + hi ---------------------------
  if constexpr (kNorm) {
    const float b = (ss[0] + ss[2]) + (ss[1] + ss[3]);  // (P[hi] + P[4 + hi]) + (P[2 + hi] + P[6 + hi])
    const float all = b + __shfl_xor(b, 32);
    if (wn == 0 && hi == 0) row_scale[RA] = rsqrtf(all / (float)K + kRmsEps);
  }

  // ---- epilogue through LDS ---------------------------------------------------------------------------------------
  auto read_c4 = [&](int row, int col) { return *reinterpret_cast<const float4*>(Cs + row * LDC + col); };
  __syncthreads();  // the stages are no longer read
#pragma unroll
  for (int r = 0; r < 16; ++r) Cs[(wm * 32 + (r >> 2) * 8 + hi * 4 + (r & 3)) * LDC + wn * 32 + r31] = acc[r];
  __syncthreads();
  epilogue_pass<bf16, EP, kNorm, BN, NT, EP == EP_RESID>(p, read_c4, row_scale, row_pos, row_page, m0, n0, 0, M, N, tid, oldc);
}

// ---- host side -------------------------------------------------------------------------------------------------
template <int AM, int EP>
static hipError_t launch_t(const GemmP& p, hipStream_t st) {
  const long tiles = (long)((p.M + BM - 1) / BM) * (p.N / BN);
  hipLaunchKernelGGL((gemm_direct64_kernel<AM, EP>), dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(NT), SMEM, st, p);
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

template <int AM, int EP>
static hipError_t raise() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_direct64_kernel<AM, EP>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)SMEM);
}

// More than 64 KB of dynamic LDS needs a one-time opt-in per kernel, outside any stream capture.
hipError_t prepare_gemm_direct64() {
  hipError_t e;
  if ((e = raise<A_ACT, EP_STORE>()) != hipSuccess) return e;
  if ((e = raise<A_ACT, EP_RESID>()) != hipSuccess) return e;
  if ((e = raise<A_NORM, EP_STORE>()) != hipSuccess) return e;
  if ((e = raise<A_NORM, EP_GELU>()) != hipSuccess) return e;
  return raise<A_NORM, EP_QKV>();
}

}  // namespace tsd
