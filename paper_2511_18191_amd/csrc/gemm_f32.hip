// fp32 GEMM: C[M,N] = A[M,K] * Wt[N,K]^T with the fused epilogues of the tiled family (gemm_epilogue.h), on the fp32 matrix
// instruction v_mfma_f32_16x16x4_f32, which adds its four products to the sum one fused multiply-add after the other in
// ascending k: the bits are those of a plain chain of fmaf over k.
//
// What bounds it: the products of fp32 handles are small (tens of rows, 64 to 512 columns), so a launch is the latency of its
// operands and a chain of K / 4 matrix instructions.  With fp32 FMAs on 4 x 4 values per lane a 64 x 64 tile read eight words of LDS
// per lane and k and LDS bandwidth bound it (40 x 64 x 256 10.7 us a launch); a matrix instruction needs two words for four k (5.8 us,
// of which the launch itself is about 4).  Eight series through tiny models: 857 us a forecast, 551 with attention's wavefront per query.
//   * TM blocks of 16 rows x 64 columns per workgroup, a wavefront per 16 columns.
//   * global -> registers (two k-tiles in flight) -> LDS (double buffered) -> MFMA -> LDS -> epilogue.
//   * LDS rows are BK + 4 words: 16-byte writes, and the fragment reads (16 rows, four consecutive k) fall on all 64 banks.
#include "tsd_internal.h"
#include "gemm_epilogue.h"
#include "tile_order.h"

namespace tsd {

typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace f32 {
constexpr int BN = 64, NT = 256, LDC = BN + 4;
template <int TM, int BK>
constexpr int tile_words() {  // two pairs of tiles, or the product
  return 2 * (16 * TM + BN) * (BK + 4) > 16 * TM * LDC ? 2 * (16 * TM + BN) * (BK + 4) : 16 * TM * LDC;
}
}  // namespace f32

template <int AM, int EP, int TM, int BK>
__global__ __launch_bounds__(f32::NT) void gemm_f32_kernel(const GemmP p) {
  using namespace f32;
  constexpr int BM = 16 * TM, LDT = BK + 4, CPR = BK / 4;  // CPR: 16-byte chunks of a tile row
  constexpr int NA = BM * CPR / NT, NB = BN * CPR / NT;
  static_assert(NA >= 1 && NB >= 1 && BK % 16 == 0 && BM * 4 <= NT, "tile");
  constexpr bool kNorm = (AM == A_NORM || AM == A_NORM32);  // RMSNorm fused as a row scale
  __shared__ __attribute__((aligned(16))) float smem[tile_words<TM, BK>()];
  __shared__ float row_scale[BM];
  __shared__ int row_pos[BM], row_page[BM];  // EP_QKV: absolute position of the row's token, its physical KV page
  float* As = smem;                 // [2][BM][LDT]
  float* Bs = smem + 2 * BM * LDT;  // [2][BN][LDT]
  float* Cs = smem;                 // [BM][LDC]
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, l15 = lane & 15, lq = lane >> 4;

  // rows of the product: fixed at launch, or capped by a device-side series count when the launch
  // is replayed from a graph while series finish (workgroups past the cap leave at once)
  const int M = p.n_dev ? min(p.M, *p.n_dev * p.nq) : p.M;
  const int N = p.N, K = p.K;
  int tm, tn;
  if (!own_tile(row_tiles<BM>(p, M), (N + BN - 1) / BN, tm, tn)) return;
  int m0 = tm * BM, m_lim = M;
  const int n0 = tn * BN;
  const float* W = reinterpret_cast<const float*>(p.W);
  if (p.tile_map) {  // routed FFN: this row tile belongs to one expert's run of slots
    const int4 tmap = reinterpret_cast<const int4*>(p.tile_map)[tm];
    m0 = tmap.y;
    m_lim = tmap.z;
    W += (long)tmap.x * p.w_stride;
  }

  // ---- loads: rows and columns past the product are clamped to the last one (their products are never stored), chunks past K
  // to the last chunk (zeroed on the way to LDS)
  const float *arow[NA], *brow[NB];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    int gm = min(m0 + (tid + i * NT) / CPR, m_lim - 1);
    if (p.src_row) gm = p.src_row[gm];
    if constexpr (AM == A_TOK) {
      int b = gm / p.nq;
      const int t = gm % p.nq;
      if (p.act) b = p.act[b];
      arow[i] = (t < p.n0) ? p.src0 + (long)b * p.stride0 + (long)t * K : p.src1 + (long)b * p.stride1 + (long)(t - p.n0) * K;
    } else {
      arow[i] = reinterpret_cast<const float*>(p.A) + (long)gm * K;
    }
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) brow[i] = W + (long)min(n0 + (tid + i * NT) / CPR, N - 1) * K;
  const int kc = tid % CPR * 4;  // (NT is a multiple of CPR: the same chunk for every load of a lane)
  static_assert(NT % CPR == 0, "chunk of a lane");
  float4 ra0[NA], rb0[NB], ra1[NA], rb1[NB];
  auto load_global = [&](int kt, float4* ra, float4* rb) {
    const int k = min(kt * BK + kc, K - 4);
#pragma unroll
    for (int i = 0; i < NA; ++i) ra[i] = *reinterpret_cast<const float4*>(arow[i] + k);
#pragma unroll
    for (int i = 0; i < NB; ++i) rb[i] = *reinterpret_cast<const float4*>(brow[i] + k);
  };
  auto store_lds = [&](int kt, int buf, const float4* ra, const float4* rb) {
    const bool in = kt * BK + kc < K;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < NA; ++i) *reinterpret_cast<float4*>(As + (buf * BM + (tid + i * NT) / CPR) * LDT + kc) = in ? ra[i] : zero;
#pragma unroll
    for (int i = 0; i < NB; ++i) *reinterpret_cast<float4*>(Bs + (buf * BN + (tid + i * NT) / CPR) * LDT + kc) = in ? rb[i] : zero;
  };

  f32x4 acc[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  // row sums of squares: per row four partial sums, one per 16-byte chunk position of a 16-wide k-run, by the lanes 4 row + position
  float ss = 0.f;
  auto compute = [&](int kt, int buf) {
    const float* at = As + (buf * BM + l15) * LDT + lq;
    const float* bt = Bs + (buf * BN + wid * 16 + l15) * LDT + lq;
    auto step = [&](int s) {
      const float b = bt[4 * s];
#pragma unroll
      for (int i = 0; i < TM; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(at[i * 16 * LDT + 4 * s], b, acc[i], 0, 0, 0);
    };
    const int left = (K - kt * BK + 3) / 4;
    if (left >= CPR) {
#pragma unroll
      for (int s = 0; s < CPR; ++s) step(s);
    } else {
      for (int s = 0; s < left; ++s) step(s);
    }
    if constexpr (kNorm) {
      if (tid < BM * 4) {
#pragma unroll
        for (int g = 0; g < BK / 16; ++g) {
          const float4 f = *reinterpret_cast<const float4*>(As + (buf * BM + (tid >> 2)) * LDT + g * 16 + (tid & 3) * 4);
          ss += f.x * f.x + f.y * f.y + f.z * f.z + f.w * f.w;
        }
      }
    }
  };

  const int nk = (K + BK - 1) / BK;
  load_global(0, ra0, rb0);
  load_global(1, ra1, rb1);
  // epilogue inputs that do not depend on the product land behind the main loop
  int2 my_meta = make_int2(0, 0);
  if constexpr (EP == EP_QKV) {
    if (tid < BM) my_meta = p.row_meta[min(m0 + tid, m_lim - 1)];
  }
  if constexpr (AM == A_TOK) {
    if (p.row_meta && tn == 0 && tid < BM) my_meta = row_meta_of(p, min(m0 + tid, m_lim - 1));
  }
  float4 oldc[TM];
  if constexpr (EP == EP_RESID) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int g = tid + i * NT, gm = min(m0 + g / (BN / 4), m_lim - 1), gn = min(n0 + (g % (BN / 4)) * 4, N - 4);
      oldc[i] = *reinterpret_cast<const float4*>(p.Cf + (long)gm * N + gn);
    }
  }
  store_lds(0, 0, ra0, rb0);
  __syncthreads();
  int kt = 0;
  // two k-tiles per trip: tile kt sits in LDS buffer 0, register set 1 holds tile kt + 1 (in flight), set 0 is free
  for (; kt + 2 < nk; kt += 2) {
    load_global(kt + 2, ra0, rb0);
    __builtin_amdgcn_sched_barrier(0);
    compute(kt, 0);
    store_lds(kt + 1, 1, ra1, rb1);
    __syncthreads();
    load_global(kt + 3, ra1, rb1);
    __builtin_amdgcn_sched_barrier(0);
    compute(kt + 1, 1);
    store_lds(kt + 2, 0, ra0, rb0);
    __syncthreads();
  }
  compute(kt, 0);
  if (kt + 1 < nk) {
    store_lds(kt + 1, 1, ra1, rb1);
    __syncthreads();
    compute(kt + 1, 1);
  }

  if constexpr (EP == EP_QKV) {
    if (tid < BM) {
      row_pos[tid] = my_meta.x;
      row_page[tid] = my_meta.y;
    }
  }
  if constexpr (AM == A_TOK) {
    if (p.row_meta && tn == 0 && tid < BM && m0 + tid < m_lim) p.row_meta[m0 + tid] = my_meta;
  }
  if constexpr (kNorm) {
    float s = ss + __shfl_xor(ss, 2);
    s += __shfl_xor(s, 1);
    if (tid < BM * 4 && (tid & 3) == 0) row_scale[tid >> 2] = rsqrtf(s / (float)K + kRmsEps);
  }
  __syncthreads();  // the tiles are no longer read
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) Cs[(i * 16 + lq * 4 + r) * LDC + wid * 16 + l15] = acc[i][r];
  __syncthreads();
  auto read_c4 = [&](int row, int col) { return *reinterpret_cast<const float4*>(Cs + row * LDC + col); };
  epilogue_pass<float, EP, kNorm, BN, NT, EP == EP_RESID, BM>(p, read_c4, row_scale, row_pos, row_page, m0, n0, 0, m_lim, N, tid, oldc);
}

// ---- host side -------------------------------------------------------------------------------------------------
template <int AM, int EP, int TM, int BK>
static hipError_t launch_shape(const GemmP& p, hipStream_t st) {
  const long tiles = (long)(p.tile_map ? p.n_mtiles : (p.M + 16 * TM - 1) / (16 * TM)) * ((p.N + f32::BN - 1) / f32::BN);
  hipLaunchKernelGGL((gemm_f32_kernel<AM, EP, TM, BK>), dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(f32::NT), 0, st, p);
  return hipGetLastError();
}

// 16-row tiles up to one per compute unit: the fewest bytes and instructions between a launch's first load and its last store.
// Beyond, 64-row tiles, which read the weights a quarter as often (64 rows / 16 rows, us, at t16 tiles of 16 rows: FFN down of K = 512
// 15.5 / 10.4 at 160, 16.0 / 16.8 at 320, 29.6 / 40.8 at 640; QKV of K = 128 11.6 / 8.4 at 240, 11.7 / 11.7 at 376, 12.5 / 16.1 at 744).
// Same bits; maps of the routed FFN are of 64 rows.
template <int AM, int EP>
static hipError_t launch_t(const GemmP& p, hipStream_t st) {
  const long t16 = (long)((p.M + 15) / 16) * ((p.N + f32::BN - 1) / f32::BN);
  return !p.tile_map && t16 <= 256 ? launch_shape<AM, EP, 1, 64>(p, st) : launch_shape<AM, EP, 4, 32>(p, st);
}

hipError_t launch_gemm_f32(int amode, int epi, const GemmP& p, hipStream_t st) {
  if (amode == A_TOK && epi == EP_STORE) return launch_t<A_TOK, EP_STORE>(p, st);
  if (amode == A_NORM && epi == EP_QKV) return launch_t<A_NORM, EP_QKV>(p, st);
  if (amode == A_ACT && epi == EP_RESID) return launch_t<A_ACT, EP_RESID>(p, st);
  if (amode == A_NORM && epi == EP_GELU) return launch_t<A_NORM, EP_GELU>(p, st);
  if (amode == A_NORM32 && epi == EP_HEAD) return launch_t<A_NORM32, EP_HEAD>(p, st);
  if (amode == A_NORM && epi == EP_STORE) return launch_t<A_NORM, EP_STORE>(p, st);
  if (amode == A_ACT && epi == EP_STORE) return launch_t<A_ACT, EP_STORE>(p, st);
  return hipErrorInvalidValue;
}

}  // namespace tsd
