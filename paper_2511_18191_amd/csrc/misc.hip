// Small kernels around the transformer pass: weight packing, prefill statistics, the fused
// acceptance / correction / commit / rollback kernel, and read-out helpers.
#include <algorithm>
#include <type_traits>

#include "accept_step.h"
#include "compact_step.h"
#include "philox.h"
#include "tsd_internal.h"

namespace tsd {

// ---- weight packing: out[n][k] = T(gain[k] * W[k][n]) ---------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void pack_kernel(const PackP p) {
  __shared__ float tile[32][33];
  const int k0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int r = ty; r < 32; r += 8) {
    int k = k0 + r, n = n0 + tx;
    float v = 0.f;
    if (k < p.K && n < p.N) v = p.W[(long)k * p.N + n] * (p.gain ? p.gain[k] : 1.f);
    tile[r][tx] = v;
  }
  __syncthreads();
  T* out = reinterpret_cast<T*>(p.out);
  for (int r = ty; r < 32; r += 8) {
    int n = n0 + r, k = k0 + tx;
    if (k < p.K && n < p.N) out[(long)n * p.K + k] = (T)tile[tx][r];
  }
}

hipError_t launch_pack(int dtype, const PackP& p, hipStream_t st) {
  dim3 grid((p.N + 31) / 32, (p.K + 31) / 32), block(256);
  if (dtype == TSD_BF16)
    hipLaunchKernelGGL(pack_kernel<bf16>, grid, block, 0, st, p);
  else
    hipLaunchKernelGGL(pack_kernel<float>, grid, block, 0, st, p);
  return hipGetLastError();
}

// ---- prefill: frozen instance statistics, normalised context, initial per-series state ------
__device__ __forceinline__ double block_sum(double v, double* sh) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += sh[i];
  return t;
}

// Every series decodes again: the active list is the identity, its count the batch, and the
// largest number of patches still needed is T.
__device__ __forceinline__ void reset_active_list(const PrefillP& p, int b) {
  if (!p.act_list) return;
  p.act_list[b] = b;
  if (b == 0) {
    p.act_count[0] = p.batch;
    p.act_count[1] = p.T;
  }
}

__device__ __forceinline__ void init_state(const PrefillP& p, int b) {
  p.len[b] = p.N - 1;  // context patches 0..N-2 are cached; patch N-1 is pending at position N-1
  p.committed[b] = 0;
  p.round[b] = 0;
  p.active[b] = 1;
  for (int i = 0; i < 5; ++i) p.stat[(long)b * 5 + i] = 0;
  reset_active_list(p, b);
}

__global__ __launch_bounds__(256) void prefill_stats_kernel(const PrefillP p) {
  __shared__ double sh[4];
  const int n = p.N * p.P;
  const int b = p.slots ? p.slots[blockIdx.x] : (int)blockIdx.x;
  const float* x = p.series + (long)blockIdx.x * n;
  double s = 0;
  for (int i = threadIdx.x; i < n; i += 256) s += x[i];
  const double mean = block_sum(s, sh) / n;
  double v = 0;
  for (int i = threadIdx.x; i < n; i += 256) {
    double dlt = x[i] - mean;
    v += dlt * dlt;
  }
  const double var = block_sum(v, sh) / n;  // population variance of the context only
  const float mf = (float)mean, sf = (float)sqrt(var + (double)kNormEps);
  float* z = p.znorm + (long)b * n;
  for (int i = threadIdx.x; i < n; i += 256) z[i] = (x[i] - mf) / sf;
  __syncthreads();
  for (int i = threadIdx.x; i < p.P; i += 256) {
    p.pending[(long)b * p.P + i] = z[(long)(p.N - 1) * p.P + i];
    p.prev[(long)b * p.P + i] = z[(long)(p.N - 2) * p.P + i];
  }
  if (threadIdx.x == 0) {
    p.mean[b] = mf;
    p.sdev[b] = sf;
    if (p.keep_counters) {  // a new series in a used slot: its draws continue the slot's round counter
      p.len[b] = p.N - 1;
      p.committed[b] = 0;
      p.active[b] = 1;
    } else {
      init_state(p, b);
    }
  }
}

__global__ __launch_bounds__(256) void reset_kernel(const PrefillP p) {
  const int b = blockIdx.x, n = p.N * p.P;
  const float* z = p.znorm + (long)b * n;
  for (int i = threadIdx.x; i < p.P; i += 256) {
    p.pending[(long)b * p.P + i] = z[(long)(p.N - 1) * p.P + i];
    p.prev[(long)b * p.P + i] = z[(long)(p.N - 2) * p.P + i];
  }
  if (threadIdx.x == 0) init_state(p, b);
}

hipError_t launch_prefill_stats(const PrefillP& p, hipStream_t st) {
  hipLaunchKernelGGL(prefill_stats_kernel, dim3(p.B), dim3(256), 0, st, p);
  return hipGetLastError();
}
hipError_t launch_reset(const PrefillP& p, hipStream_t st) {
  hipLaunchKernelGGL(reset_kernel, dim3(p.B), dim3(256), 0, st, p);
  return hipGetLastError();
}

// ---- acceptance + correction + commit + rollback ---------------------------------------------
// Sampled proposals: X[b, i-1, :] = mu_q[b, i-1, :] + sigma_q * eps for the covered series, with
// each series' own round counter.  One 64-thread block per series.
__global__ __launch_bounds__(64) void sample_kernel(const SampleP p) {
  if (p.n_dev && (int)blockIdx.x >= *p.n_dev) return;
  const int b = p.act ? p.act[blockIdx.x] : (int)blockIdx.x;
  const unsigned r = (unsigned)p.round[b];
  const long off = ((long)b * p.K + (p.i - 1)) * p.P;
  for (int e = threadIdx.x; e < p.P; e += 64)
    p.X[off + e] = p.mu_q[off + e] + (p.sigma_q_vec ? p.sigma_q_vec[e] : p.sigma_q) * normal_draw((unsigned)b, r, (unsigned)p.i, kStreamProposal, e, p.key0, p.key1);
}
hipError_t launch_sample(const SampleP& p, hipStream_t st) {
  if (p.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(sample_kernel, dim3(p.n), dim3(64), 0, st, p);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void accept_kernel(const AcceptP p) { accept_step(p); }

hipError_t launch_accept(const AcceptP& p, hipStream_t st) {
  hipLaunchKernelGGL(accept_kernel, dim3(p.B), dim3(256), 0, st, p);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void row_meta_kernel(const GemmP p) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < p.M) p.row_meta[i] = row_meta_of(p, i);
}
hipError_t launch_row_meta(const GemmP& p, hipStream_t st) {
  hipLaunchKernelGGL(row_meta_kernel, dim3((unsigned)((p.M + 255) / 256)), dim3(256), 0, st, p);
  return hipGetLastError();
}

__global__ void fill_int_kernel(int* p, int value, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = value;
}
hipError_t launch_fill_int(int* p, int value, int n, hipStream_t st) {
  hipLaunchKernelGGL(fill_int_kernel, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, st, p, value, n);
  return hipGetLastError();
}

// ---- read-out helpers ------------------------------------------------------------------------
__global__ void forecast_out_kernel(const float* forecast, const float* mean, const float* sdev, const int* committed,
                                    float* out, int P, int T, int H) {
  const int b = blockIdx.x;
  const int have = committed[b] * P;
  for (int t = threadIdx.x; t < H; t += blockDim.x)
    out[(long)b * H + t] = t < have ? forecast[(long)b * T * P + t] * sdev[b] + mean[b] : 0.f;
}
hipError_t launch_forecast_out(const float* forecast, const float* mean, const float* sdev, const int* committed,
                               float* out, int B, int P, int T, int H, hipStream_t st) {
  hipLaunchKernelGGL(forecast_out_kernel, dim3(B), dim3(256), 0, st, forecast, mean, sdev, committed, out, P, T, H);
  return hipGetLastError();
}

// One block: stable compaction of the active series (ascending series index) and their count.
// count[0] = number of active series, count[1] = the largest number of patches any of them still
// needs (T - committed).
__global__ __launch_bounds__(1024) void compact_active_kernel(const int* active, const int* committed, int T, int B,
                                                              int* list, int* count, int* host) {
  const int2 now = compact_step<16>(active, committed, T, B, list, [](const int* a) { return *a; });
  if (threadIdx.x == 0) {
    count[0] = now.x;
    count[1] = now.y;
    if (host) {
      // straight into pinned host memory, so the caller needs neither a copy nor a stream wait: it watches
      // host[2] for this launch's number, which is stored last
      const int seq = count[4] + 1;
      count[4] = seq;
      host[0] = now.x;
      host[1] = now.y;
      __hip_atomic_store(&host[2], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}
hipError_t launch_compact_active(const int* active, const int* committed, int T, int B, int* list, int* count,
                                 int* host, hipStream_t st) {
  hipLaunchKernelGGL(compact_active_kernel, dim3(1), dim3(1024), 0, st, active, committed, T, B, list, count, host);
  return hipGetLastError();
}

__global__ void sum_stats_kernel(const long long* stat, int B, long long* out5) {
  long long c[5] = {0, 0, 0, 0, 0};
  for (int i = threadIdx.x; i < B; i += 64)
    for (int j = 0; j < 5; ++j) c[j] += stat[(long)i * 5 + j];
  for (int j = 0; j < 5; ++j) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) c[j] += __shfl_xor(c[j], o);
    if (threadIdx.x == 0) out5[j] = c[j];
  }
}
__global__ void identity_list_kernel(int* list, int* count, int B, int T) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < B) list[b] = b;
  if (b == 0) {
    count[0] = B;
    count[1] = T;
  }
}
hipError_t launch_identity_list(int* list, int* count, int B, int T, hipStream_t st) {
  hipLaunchKernelGGL(identity_list_kernel, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, st, list, count, B, T);
  return hipGetLastError();
}

hipError_t launch_sum_stats(const long long* stat, int B, long long* out5, hipStream_t st) {
  hipLaunchKernelGGL(sum_stats_kernel, dim3(1), dim3(64), 0, st, stat, B, out5);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void copy_kernel(uint4* dst, const uint4* src, size_t n16) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}
hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t st) {
  const size_t n16 = bytes / 16;
  const unsigned grid = (unsigned)std::min<size_t>((n16 + 255) / 256, 256 * 32);
  hipLaunchKernelGGL(copy_kernel, dim3(grid), dim3(256), 0, st, (uint4*)dst, (const uint4*)src, n16);
  return hipGetLastError();
}

// Matrix-core tap: four independent accumulation chains per wavefront keep the MFMA pipe full; the
// operands stay in registers, so nothing but the matrix cores is measured.
__global__ __launch_bounds__(256) void mfma_peak_kernel(int iters, float* sink) {
  bf16x8 a, b;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    a[e] = (bf16)(0.015625f * (float)(1 + ((threadIdx.x + e) & 3)));
    b[e] = (bf16)(0.015625f * (float)(1 + ((threadIdx.x >> 2) & 3)));
  }
  f32x16 c0, c1, c2, c3;
#pragma unroll
  for (int r = 0; r < 16; ++r) c0[r] = c1[r] = c2[r] = c3[r] = 0.f;
  for (int it = 0; it < iters; ++it) {
    c0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c1, 0, 0, 0);
    c2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c2, 0, 0, 0);
    c3 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c3, 0, 0, 0);
  }
  float s = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) s += c0[r] + c1[r] + c2[r] + c3[r];
  sink[(size_t)blockIdx.x * 256 + threadIdx.x] = s;
}
hipError_t launch_mfma_peak(int blocks, int iters, float* sink, hipStream_t st) {
  hipLaunchKernelGGL(mfma_peak_kernel, dim3(blocks), dim3(256), 0, st, iters, sink);
  return hipGetLastError();
}

__global__ void fill_nan_kernel(float* p, long n) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = NAN;
}
hipError_t launch_fill_nan(float* p, long n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_nan_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n);
  return hipGetLastError();
}

}  // namespace tsd
