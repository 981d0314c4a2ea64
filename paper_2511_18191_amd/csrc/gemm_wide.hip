// Wide-tile bf16 GEMM for products of more than one 64 x 64 tile per compute unit: C[M,N] = A[M,K] * Wt[N,K]^T with the
// fused epilogues of the tiled family.  Operands go from global memory straight into LDS as in gemm_direct64.hip (stages of
// whole rows, swizzled chunks, one barrier per k-tile, the same order of sums: same bits), tiles are as large as the
// product's tile count allows.
//
// What bounds the largest tile (256 x 256, eight wavefronts of 64 x 128, one workgroup per compute unit; 16384x4096x1024 without
// its epilogue): MFMAs alone take 57 us, 77 with the RMSNorm row sums on the A fragments, 82 with the fragment reads from LDS;
// the loads alone take 40 (62 where the weights come from HBM); together 113.  So neither path is at its limit, what costs is
// where one waits for the other:
//   * A compute unit takes in 64 bytes per clock, a 64 KB stage 1024 clocks, and a wavefront stands still until its loads are
//     accepted.  Issued in one batch behind the barrier they kept the matrix cores idle meanwhile; so a wavefront's loads of a
//     stage are spread among the MFMAs of two sub-steps (119 -> 113 us).
//   * The MFMAs take the weights as first operand and the rows as second: a lane then holds four consecutive columns of ONE row
//     (register 4 q + e of a 32 x 32 block: column 8 q + 4 (lane / 32) + e of row lane % 32).  The row scale is one value per lane that
//     never goes through LDS, rotary partners sit in the same lane, GELU and the packing to bf16 happen in registers, and the
//     results pass through a patch of LDS of the wavefront's own (the stages it no longer needs) as 16-byte pieces, to leave as whole
//     cache lines: one barrier in the whole epilogue.  (Through LDS in fp32, 64 rows of the tile at a time: 40 us more per launch.)
// Products of a context pass of 16343 rows, before (128 x 128 tiles) / now, us: 16343x4096x1024 GELU 183 / 144, 16343x3072x1024
// QKV 133 / 116, 16343x1024x4096 residual 142 / 131; of a verification pass: 7168x4096x1024 75 / 67, 7168x3072x1024 66 / 60,
// 7168x1024x4096 69 / 63.
#include "direct_lds.h"
#include "gemm_epilogue.h"
#include "tile_order.h"

namespace tsd {

// BM x BN x BK tiles, WGM x WGN wavefronts of TM x TN blocks of 32 x 32, NS stages
template <int BM_, int BN_, int BK_, int WGM_, int WGN_, int NS_>
struct WideShape {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, WGM = WGM_, WGN = WGN_, NS = NS_;
  static constexpr int NW = WGM * WGN, NT = NW * 64;
  static constexpr int ROWB = BK * 2;                    // bytes of a stage row: 64 or 128
  static constexpr int CPR = ROWB / 16;                  // 16-byte chunks per row
  static constexpr int RPL = 1024 / ROWB;                // rows a load instruction covers
  static constexpr int STAGE = (BM + BN) * ROWB;
  static constexpr int NL = STAGE / 1024 / NW;           // load instructions of a wavefront per stage
  static constexpr int FIRST = NL / 2;                   // ... of which this many go with the sub-step behind the barrier
  static constexpr int REGION = NL * 1024;               // a wavefront's bytes of a stage
  static constexpr int BIAS = REGION / 2 / 1024 * 1024;  // M0 points here inside the region: immediates stay small
  static constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32;
  static constexpr int NSUB = BK / 16;                   // k16 sub-steps per k-tile
  static constexpr int NPAR = 64 / BK;                   // k-tiles per 64-wide k-run
  static constexpr int PATCH = NS * STAGE / NW / 1024 * 1024;  // a wavefront's share of the stages, for its results
  static constexpr size_t SMEM = (size_t)NS * STAGE + BM * 8;  // stages, then row_pos / row_page
  static_assert(BK == 32 || BK == 64, "k-tiles of 32 or 64");
  static_assert(STAGE % (1024 * NW) == 0 && BM % RPL == 0, "every wavefront loads whole instructions, each all A or all B");
  static_assert(REGION - BIAS <= 4096 && BIAS <= 4096, "immediate offsets are 13 bits, signed");
  static_assert(NPAR == 1 || NS % 2 == 1, "the loop over pairs of 32-wide k-tiles is written for an odd number of stages");
  static_assert(SMEM <= 160 * 1024, "LDS of a compute unit");
};

// The MFMAs of a sub-step (from number m on) with the loads LO .. HI - 1 spread evenly among them.
template <int m, int TM, int TN, int LO, int HI, int BIAS>
__device__ __forceinline__ void mfma_steps(f32x16 (*acc)[TN], const bf16x8* af, const bf16x8* bfr, const bf16* const* gp, long koff,
                                           void __attribute__((address_space(3)))* base) {
  // PER loads go with every EVERY-th MFMA, G before this one
  constexpr int NM = TM * TN, NLD = HI - LO, PER = (NLD + NM - 1) / NM, EVERY = NLD > 0 ? NM * PER / NLD : NM + 1, G = m / EVERY * PER;
  if constexpr (m < NM) {
    constexpr int i = m / TN, j = m % TN;
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
    if constexpr (NLD > 0 && m % EVERY == EVERY - 1 && G < NLD) {
      __builtin_amdgcn_sched_barrier(0);
      issue_loads<LO + G, (LO + G + PER < HI ? LO + G + PER : HI), BIAS>(gp, koff, base);
      __builtin_amdgcn_sched_barrier(0);
    }
    mfma_steps<m + 1, TM, TN, LO, HI, BIAS>(acc, af, bfr, gp, koff, base);
  }
}

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  const bf16x2 v = {(bf16)a, (bf16)b};
  return __builtin_bit_cast(unsigned, v);
}
__device__ __forceinline__ uint2 pack_bf16(const float* v) { return make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])); }

template <int AM, int EP, typename S>
__global__ __launch_bounds__(S::NT, 2) void gemm_wide_kernel(const GemmP p) {
  constexpr bool kNorm = (AM == A_NORM);
  constexpr int BM = S::BM, BN = S::BN, BK = S::BK, NS = S::NS, TM = S::TM, TN = S::TN, NL = S::NL, REGION = S::REGION,
                STAGE = S::STAGE, BIAS = S::BIAS, ROWB = S::ROWB, CPR = S::CPR, RPL = S::RPL, NSUB = S::NSUB, NPAR = S::NPAR, WGN = S::WGN;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int* row_pos = reinterpret_cast<int*>(smem + NS * STAGE);  // [BM] EP_QKV
  int* row_page = row_pos + BM;                              // [BM] EP_QKV

  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wid / WGN, wn = wid % WGN;
  // rows of the product: fixed at launch, or capped by a device-side series count (workgroups past the cap leave)
  const int M = p.n_dev ? min(p.M, *p.n_dev * p.nq) : p.M;
  const int N = p.N, K = p.K;
  int tm, tn;
  if (!own_tile(row_tiles<BM>(p, M), N / BN, tm, tn)) return;
  int m0 = tm * BM, m_lim = M;
  const int n0 = tn * BN;
  const bf16* Wp = reinterpret_cast<const bf16*>(p.W);
  if (p.tile_map) {  // routed FFN: this row tile belongs to one expert's run of slots
    const int4 tmap = reinterpret_cast<const int4*>(p.tile_map)[tm];
    m0 = tmap.y;
    m_lim = tmap.z;
    Wp += (long)tmap.x * p.w_stride;
  }
  const int r31 = lane & 31, hi = lane >> 5;

  // (requested before the operands: loads return in order, so nothing older than the stages' loads disturbs their counted waits)
  int2 my_meta = make_int2(0, 0);
  if constexpr (EP == EP_QKV) {
    static_assert(BM <= S::NT, "one row per lane");
    my_meta = p.row_meta[min(m0 + min(tid, BM - 1), m_lim - 1)];
  }

  // ---- loads (see gemm_direct64.hip): wavefront w fills the stage rows [NL * RPL * w, NL * RPL * (w + 1))
  auto swizzle = [](int R) { return BK == 64 ? (R >> 1) & 7 : (R >> 2) & 3; };
  const bf16* Ap = reinterpret_cast<const bf16*>(p.A);
  const bf16* gp[NL];
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const int R = (wid * NL + j) * RPL + lane / CPR;
    const int chunk = (lane % CPR) ^ swizzle(R);
    const bf16* row;
    if ((wid * NL + j) * RPL < BM) {  // (uniform per instruction)
      int gm = min(m0 + R, m_lim - 1);  // rows past the end are clamped: their products are never stored
      if (p.src_row) gm = p.src_row[gm];
      row = Ap + (long)gm * K;
    } else {
      row = Wp + (long)(n0 + R - BM) * K;
    }
    gp[j] = row + chunk * 8 - (j * 1024 - BIAS) / 2;
  }
  auto stage_base = [&](int kt) { return TSD_LDS_PTR(smem + (kt % NS) * STAGE + wid * REGION + BIAS); };

  // Long contractions of activations are summed in four runs of ceil(nk / 4) k-tiles, each from zero, the runs added in
  // order (the order of the split workgroups of gemm.hip, which every kernel that can take such a product keeps to).  The running
  // sum takes as many registers as the accumulators: wavefronts of 64 x 64 at most.
  constexpr bool kQuarters = AM == A_ACT && TM * TN <= 4 && BK == 64;
  f32x16 tot[kQuarters ? TM : 1][kQuarters ? TN : 1];
  f32x16 acc[TM][TN];
  const f32x16 zero = {};
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  float ss[TM][4];  // row-sum chains of this lane: chunk positions hi, 2 + hi, 4 + hi, 6 + hi of a 64-wide k-run
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int c = 0; c < 4; ++c) ss[i][c] = 0.f;
  int offA[TM], offB[TN], swA[TM], swB[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int R = wm * (TM * 32) + i * 32 + r31;
    offA[i] = R * ROWB;
    swA[i] = swizzle(R);
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int R = BM + wn * (TN * 32) + j * 32 + r31;
    offB[j] = R * ROWB;
    swB[j] = swizzle(R);
  }

  // The k loop is software-pipelined by k16 sub-steps: while the MFMAs of one run, the fragments of the next are on their way from LDS, also
  // across k-tiles (two sets in turn).  One bare barrier per k-tile, before its LAST sub-step: this wavefront's loads of k-tile kt + 1 are
  // done then and its fragments of k-tile kt all sit in registers, so behind it k-tile kt + 1 can be read and the slot of k-tile kt refilled.
  bf16x8 fa[2][TM], fb[2][TN];
  auto read_frags = [&](int kt, int s, bf16x8* af, bf16x8* bfr) {
    const unsigned char* st = smem + (kt % NS) * STAGE;
#pragma unroll
    for (int i = 0; i < TM; ++i) af[i] = *reinterpret_cast<const bf16x8*>(st + offA[i] + (((2 * s + hi) ^ swA[i]) << 4));
#pragma unroll
    for (int j = 0; j < TN; ++j) bfr[j] = *reinterpret_cast<const bf16x8*>(st + offB[j] + (((2 * s + hi) ^ swB[j]) << 4));
  };
  auto row_sums = [&](auto cpos, const bf16x8* af) {
    constexpr int C = decltype(cpos)::value;
    if constexpr (kNorm) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bf16x2 pr = {af[i][2 * e], af[i][2 * e + 1]};
          ss[i][C] = __builtin_amdgcn_fdot2_f32_bf16(pr, pr, ss[i][C], false);
        }
    }
  };
  // (an empty statement that makes the compiler wait for a fragment set before the next set's reads are issued)
  auto arrived = [&](bf16x8* af, bf16x8* bfr) {
#pragma unroll
    for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(af[i]));
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(bfr[j]));
  };
  // One k-tile.  PAR: its position inside the 64-wide k-run; PEND: the loads this wavefront may leave in flight at the barrier, or -1
  // for the last k-tile (no barrier); REFILL: k-tile kt + NS exists, the first loads for it go with the sub-step behind the barrier;
  // RPREV: so does k-tile kt - 1 + NS, whose other loads go with this k-tile's first sub-step.
  constexpr int FIRST = S::FIRST;
  auto tile = [&](auto par, int kt, auto pend, auto refill, auto rprev) {
    constexpr int PAR = decltype(par)::value, PEND = decltype(pend)::value;
    constexpr bool REFILL = decltype(refill)::value != 0, RPREV = decltype(rprev)::value != 0;
    const auto sub = [&](auto sc) {
      constexpr int s = decltype(sc)::value;
      arrived(fa[s & 1], fb[s & 1]);
      if constexpr (s + 1 < NSUB) {
        read_frags(kt, s + 1, fa[(s + 1) & 1], fb[(s + 1) & 1]);
      } else if constexpr (PEND >= 0) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(PEND) : "memory");
        read_frags(kt + 1, 0, fa[(s + 1) & 1], fb[(s + 1) & 1]);
      }
      __builtin_amdgcn_sched_barrier(0);
      row_sums(IC<PAR * NSUB + s>{}, fa[s & 1]);
      if constexpr (s == NSUB - 1 && REFILL)
        mfma_steps<0, TM, TN, 0, FIRST, BIAS>(acc, fa[s & 1], fb[s & 1], gp, (long)(kt + NS) * BK, stage_base(kt));
      else if constexpr (s == 0 && RPREV)
        mfma_steps<0, TM, TN, FIRST, NL, BIAS>(acc, fa[s & 1], fb[s & 1], gp, (long)(kt - 1 + NS) * BK, stage_base(kt - 1));
      else
        mfma_steps<0, TM, TN, 0, 0, BIAS>(acc, fa[s & 1], fb[s & 1], gp, 0, nullptr);
      __builtin_amdgcn_sched_barrier(0);
    };
    sub(IC<0>{});
    sub(IC<1>{});
    if constexpr (NSUB == 4) {
      sub(IC<2>{});
      sub(IC<3>{});
    }
  };

  // ---- main loop (K is a multiple of 64 and more than NS k-tiles) ---------------------------------------------------------
  const int nk = K / BK;
#pragma unroll
  for (int s = 0; s < NS; ++s) issue_loads<0, NL, BIAS>(gp, (long)s * BK, stage_base(s));
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 1) * NL) : "memory");
  read_frags(0, 0, fa[0], fb[0]);
  constexpr int STEADY_PEND = (NS - 2) * NL;
  const int n_steady = nk - NS;
  const bool quarters = kQuarters && K >= kQuarterK;
  const int run = (nk + 3) / 4;
  auto fold = [&](int done) {  // `done` k-tiles are in acc: at a run's end move them into the running sum
    if constexpr (kQuarters) {
      if (!quarters || done % run != 0 || done >= nk) return;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
        {
          tot[i][j] = done == run ? acc[i][j] : tot[i][j] + acc[i][j];
          acc[i][j] = zero;
        }
    }
  };
  tile(IC<0>{}, 0, IC<STEADY_PEND>{}, IC<1>{}, IC<0>{});
  int kt = 1;
  if constexpr (NPAR == 1) {
    for (; kt < n_steady; ++kt) {
      fold(kt);
      tile(IC<0>{}, kt, IC<STEADY_PEND>{}, IC<1>{}, IC<1>{});
    }
  } else {
    for (; kt + 1 < n_steady; kt += 2) {  // (nk is even, nk - NS odd)
      tile(IC<1>{}, kt, IC<STEADY_PEND>{}, IC<1>{}, IC<1>{});
      tile(IC<0>{}, kt + 1, IC<STEADY_PEND>{}, IC<1>{}, IC<1>{});
    }
  }
  // tail: k-tile nk - NS + t leaves NS - 2 - t stages in flight at its barrier; the last one has no barrier
  auto tail = [&](auto self, auto tc) {
    constexpr int t = decltype(tc)::value;
    fold(kt + t);
    constexpr int PARI = NPAR == 1 ? 0 : (t + 1) & 1;
    if constexpr (t + 1 < NS) {
      tile(IC<PARI>{}, kt + t, IC<(NS - 2 - t) * NL>{}, IC<0>{}, IC<(t == 0 ? 1 : 0)>{});
      self(self, IC<t + 1>{});
    } else {
      tile(IC<PARI>{}, kt + t, IC<-1>{}, IC<0>{}, IC<(t == 0 ? 1 : 0)>{});
    }
  };
  tail(tail, IC<0>{});
  if constexpr (kQuarters) {
    if (quarters) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = tot[i][j] + acc[i][j];
    }
  }

  // ---- epilogue ---------------------------------------------------------------------------------------------------------
  if constexpr (EP == EP_QKV) {
    if (tid < BM) {
      row_pos[tid] = my_meta.x;
      row_page[tid] = my_meta.y;
    }
  }
  float rs[TM];  // RMSNorm scale of this lane's row of block i
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    rs[i] = 1.f;
    if constexpr (kNorm) {
      const float b = (ss[i][0] + ss[i][2]) + (ss[i][1] + ss[i][3]);  // (P[hi] + P[4 + hi]) + (P[2 + hi] + P[6 + hi])
      rs[i] = rsqrtf((b + __shfl_xor(b, 32)) / (float)K + kRmsEps);
    }
  }
  constexpr int CW = TN * 32;  // columns of a wavefront
  const int mw = wm * (TM * 32), gn0 = n0 + wn * CW;
  unsigned char* patch = smem + wid * S::PATCH;
  auto wave_order = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  if constexpr (EP == EP_GELU || EP == EP_QKV) {
    __syncthreads();  // the stages are no longer read; from here on every wavefront is on its own
    // A row of the wavefront's results is RB bytes of bf16.  Its 16-byte chunk c sits at c ^ (row mod the chunks of a row), the two
    // halves of a chunk change places every eight rows: the 8-byte writes of 16 rows then fall on all banks.
    constexpr int RB = CW * 2, CM = RB / 16 - 1;
    static_assert(TN == 2 || TN == 4, "rows of 128 or 256 bytes");
    static_assert(TM * 32 * RB <= S::PATCH, "results fit the wavefront's share of the stages");
    auto put = [&](int i, int j, int q, const float* v) {  // columns 32 j + 8 q + 4 hi .. + 3 of row 32 i + r31
      *reinterpret_cast<uint2*>(patch + (i * 32 + r31) * RB + (((j * 4 + q) ^ (r31 & CM)) << 4) + ((hi ^ ((r31 >> 3) & 1)) << 3)) = pack_bf16(v);
    };
    if constexpr (EP == EP_GELU) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = gelu_tanh(acc[i][j][4 * q + e] * rs[i]);
            put(i, j, q, v);
          }
    } else {
      // RoPE turns dims d and d + HD / 2 of a head against each other: blocks j and j + 1 (head_dim 64), or groups q and q + 2 (32) or
      // q + 1 (16) of a block, of the same lane
      auto rotate = [&](auto hdc) {
        constexpr int HD = decltype(hdc)::value, DJ = HD == 64 ? 1 : 0, DQ = HD == 64 ? 0 : HD / 16;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const long tab = (long)row_pos[mw + i * 32 + r31] * (HD / 2) + 4 * hi;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (DQ && (q & DQ)) continue;
            const int f = HD == 64 ? 8 * q : 8 * (q & (DQ - 1));
            const float4 c4 = *reinterpret_cast<const float4*>(p.rope_cos + tab + f), s4 = *reinterpret_cast<const float4*>(p.rope_sin + tab + f);
            const float cs[4] = {c4.x, c4.y, c4.z, c4.w}, sn[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
            for (int j = 0; j < TN; j += 1 + DJ) {
              const bool turn = gn0 + j * 32 < 2 * p.D;  // queries and keys
              float lo[4], up[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const float a = acc[i][j][4 * q + e] * rs[i], b = acc[i][j + DJ][4 * (q + DQ) + e] * rs[i];
                lo[e] = turn ? a * cs[e] - b * sn[e] : a;
                up[e] = turn ? b * cs[e] + a * sn[e] : b;
              }
              put(i, j, q, lo);
              put(i, j + DJ, q + DQ, up);
            }
          }
        }
      };
      if (TN == 4 || p.hd == 64) rotate(IC<64>{});  // (the launcher gives other head sizes to shapes with TN = 2)
      else if (p.hd == 32) rotate(IC<32>{});
      else rotate(IC<16>{});
    }
    wave_order();
    constexpr int LPR = RB / 16, RPI = 64 / LPR;  // lanes per row, rows per instruction
    const int rl = lane / LPR, ch = lane % LPR;
    const int gn = gn0 + ch * 8;
    int which = 0, c = 0, head = 0, dim = 0;
    if constexpr (EP == EP_QKV) {
      which = gn / p.D;
      c = gn - which * p.D;
      head = c / p.hd;
      dim = c - head * p.hd;
    }
#pragma unroll
    for (int t = 0; t < TM * 32 / RPI; ++t) {
      const int row = RPI * t + rl;
      uint4 v = *reinterpret_cast<const uint4*>(patch + row * RB + ((ch ^ (row & CM)) << 4));
      if ((RPI * t >> 3) & 1) v = make_uint4(v.z, v.w, v.x, v.y);
      const int gm = m0 + mw + row;
      if (gm >= m_lim) continue;
      if constexpr (EP == EP_GELU) {
        *reinterpret_cast<uint4*>(reinterpret_cast<bf16*>(p.Ct) + (long)gm * N + gn) = v;
      } else if (which == 0) {
        *reinterpret_cast<uint4*>(reinterpret_cast<bf16*>(p.q_out) + (long)gm * p.D + c) = v;
      } else {
        const int tok = row_pos[mw + row] & (p.PT - 1);
        const long off = ((((long)row_page[mw + row] * 2 + (which - 1)) * p.Hh + head) * p.PT + tok) * p.hd + dim;
        *reinterpret_cast<uint4*>(reinterpret_cast<bf16*>(p.kv_pool) + off) = v;
      }
    }
  } else {
    // fp32 rows, 32 at a time; chunk c of a row at c ^ (row mod 8)
    static_assert(32 * CW * 4 <= S::PATCH, "32 rows fit the wavefront's share of the stages");
    constexpr int LPR = CW / 4;       // lanes per row
    constexpr int RPI = 64 / LPR;     // rows per instruction
    constexpr int NI = 32 / RPI, NB = NI < 8 ? NI : 8;  // instructions of a block row; old values fetched ahead
    const int ch = lane % LPR, rl = lane / LPR, gn = gn0 + ch * 4;
    float4 old[2][NB];  // the old residual, requested a batch ahead
    auto row_of = [&](int b, int t) { return mw + b * (NB * RPI) + t * RPI + rl; };
    auto fetch = [&](int b) {  // b: batch of NB instructions
      if constexpr (EP == EP_RESID) {
#pragma unroll
        for (int t = 0; t < NB; ++t) {
          const int gm = min(m0 + row_of(b, t), m_lim - 1);
          old[b & 1][t] = *reinterpret_cast<const float4*>(p.Cf + (long)gm * N + gn);
        }
      }
    };
    fetch(0);
    __syncthreads();  // the stages are no longer read; from here on every wavefront is on its own
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if (i > 0) wave_order();
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c = (j * 8 + 2 * q + hi) ^ (r31 & 7);
          *reinterpret_cast<float4*>(patch + r31 * (CW * 4) + (c << 4)) =
              make_float4(acc[i][j][4 * q] * rs[i], acc[i][j][4 * q + 1] * rs[i], acc[i][j][4 * q + 2] * rs[i], acc[i][j][4 * q + 3] * rs[i]);
        }
      wave_order();
#pragma unroll
      for (int h = 0; h < NI / NB; ++h) {
        const int b = i * (NI / NB) + h;
        if (b + 1 < TM * (NI / NB)) fetch(b + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < NB; ++t) {
          const int row = (h * NB + t) * RPI + rl;
          float4 v = *reinterpret_cast<const float4*>(patch + row * (CW * 4) + ((ch ^ (row & 7)) << 4));
          if constexpr (EP == EP_RESID) {
            v.x = old[b & 1][t].x + v.x;
            v.y = old[b & 1][t].y + v.y;
            v.z = old[b & 1][t].z + v.z;
            v.w = old[b & 1][t].w + v.w;
          }
          const int gm = m0 + row_of(b, t);
          if (gm < m_lim) {
            *reinterpret_cast<float4*>(p.Cf + (long)gm * N + gn) = v;
            if (p.Cb) store4<bf16>(reinterpret_cast<bf16*>(p.Cb) + (long)gm * N + gn, v);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}

// ---- host side -------------------------------------------------------------------------------------------------
using Wide256 = WideShape<256, 256, 64, 4, 2, 2>;     // eight wavefronts of 64 x 128, one workgroup per compute unit
using Wide128x256 = WideShape<128, 256, 32, 2, 2, 3>; // four of 64 x 128, two workgroups
using Wide256x128 = WideShape<256, 128, 64, 4, 2, 3>; // eight of 64 x 64, one workgroup
using Wide128 = WideShape<128, 128, 64, 2, 2, 2>;     // four of 64 x 64, two workgroups
using Wide128Deep = WideShape<128, 128, 64, 2, 2, 3>; // ... one workgroup
using Wide128x64 = WideShape<128, 64, 64, 4, 1, 2>;   // four of 32 x 64, three workgroups
using Wide128x64Deep = WideShape<128, 64, 64, 4, 1, 3>;  // ... two workgroups

DirectTile gemm_direct_tile(int dtype, int amode, int epi, const GemmP& p) {
  if (dtype != TSD_BF16 || p.no_wide) return kTileNone;
  if (!p.tile_map && (p.src_row || p.force_bm)) return kTileNone;
  return direct_tile(amode, epi, p.M, p.N, p.K, p.hd, p.tile_map ? p.force_bm : 0, p.parts && p.Cb);
}

template <int AM, int EP, typename S>
static hipError_t launch_shape(const GemmP& p, hipStream_t st) {
  const long tiles = (long)(p.tile_map ? p.n_mtiles : (p.M + S::BM - 1) / S::BM) * (p.N / S::BN);
  hipLaunchKernelGGL((gemm_wide_kernel<AM, EP, S>), dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(S::NT), S::SMEM, st, p);
  return hipGetLastError();
}

template <int AM, int EP>
static hipError_t launch_tile(DirectTile tile, const GemmP& p, hipStream_t st) {
  if constexpr (has_direct_kernel(AM, EP, kTile256x128)) {
    if (tile == kTile256x128) return launch_shape<AM, EP, Wide256x128>(p, st);
  }
  if constexpr (has_direct_kernel(AM, EP, kTile256)) {
    if (tile == kTile256) return launch_shape<AM, EP, Wide256>(p, st);
  }
  if constexpr (has_direct_kernel(AM, EP, kTile128x256)) {
    if (tile == kTile128x256) return launch_shape<AM, EP, Wide128x256>(p, st);
  }
  if constexpr (has_direct_kernel(AM, EP, kTile128x64)) {
    if (tile == kTile128x64) {
      const long t = (long)((p.M + 127) / 128) * (p.N / 64);
      return t <= 512 && p.K >= 256 ? launch_shape<AM, EP, Wide128x64Deep>(p, st) : launch_shape<AM, EP, Wide128x64>(p, st);
    }
  }
  if (tile != kTile128) return hipErrorInvalidValue;
  if constexpr (AM == A_ACT) {
    const long t128 = (long)((p.M + 127) / 128) * (p.N / 128);
    if (!p.tile_map && t128 <= 256 && p.K >= 256) return launch_shape<AM, EP, Wide128Deep>(p, st);
  }
  return launch_shape<AM, EP, Wide128>(p, st);
}

hipError_t launch_gemm_wide(int amode, int epi, DirectTile tile, const GemmP& p, hipStream_t st) {
  if (amode == A_ACT && epi == EP_STORE) return launch_tile<A_ACT, EP_STORE>(tile, p, st);
  if (amode == A_ACT && epi == EP_RESID) return launch_tile<A_ACT, EP_RESID>(tile, p, st);
  if (amode == A_NORM && epi == EP_STORE) return launch_tile<A_NORM, EP_STORE>(tile, p, st);
  if (amode == A_NORM && epi == EP_GELU) return launch_tile<A_NORM, EP_GELU>(tile, p, st);
  if (amode == A_NORM && epi == EP_QKV) return launch_tile<A_NORM, EP_QKV>(tile, p, st);
  return hipErrorInvalidValue;
}

// More than 64 KB of dynamic LDS needs a one-time opt-in per kernel, outside any stream capture.
template <int AM, int EP, typename... S>
static hipError_t raise() {
  hipError_t e = hipSuccess;
  ((e = e != hipSuccess ? e
                        : hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_wide_kernel<AM, EP, S>),
                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::SMEM)),
   ...);
  return e;
}

hipError_t prepare_gemm_wide() {
  hipError_t e;
  if ((e = raise<A_ACT, EP_STORE, Wide256x128, Wide128, Wide128Deep>()) != hipSuccess) return e;
  if ((e = raise<A_ACT, EP_RESID, Wide256x128, Wide128, Wide128Deep>()) != hipSuccess) return e;
  if ((e = raise<A_NORM, EP_STORE, Wide128>()) != hipSuccess) return e;
  if ((e = raise<A_NORM, EP_GELU, Wide256, Wide128, Wide128x64, Wide128x64Deep>()) != hipSuccess) return e;
  return raise<A_NORM, EP_QKV, Wide256, Wide128x256, Wide128, Wide128x64, Wide128x64Deep>();
}

}  // namespace tsd
