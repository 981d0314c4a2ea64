// tsd_accept_commit_static: the acceptance / correction / commit step of one round on caller tensors, for
// callers that cannot allocate device memory (code under HIP graph capture, tight serving loops, harnesses
// that forbid it).  It runs the same accept_kernel as tsd_accept_commit, which without a handle keeps no state: one launch (a
// kernel that first set up per-series state in a device array took 2 of the step's 10 us).  Only the synchronised round's
// minimum lives in a file-scope device word.
#include <climits>
#include <cmath>
#include <cstring>
#include <string>

#include "tsd_internal.h"

namespace tsd {
// implemented in tsd_api.hip: records the message tsd_last_error(NULL) returns
int fail_no_handle(int code, const std::string& msg);
}  // namespace tsd

using namespace tsd;

namespace {

// Limits of the static variant.
constexpr int kMaxB = 4096;             // series per call
constexpr int kMaxK = 16;               // proposals per round
constexpr long kMaxBP = 256 * 1024;     // B * P: e.g. 1024 series of 256-step patches, or 4096 of 64

static __device__ int sync_word;

// Address of this device's copy of `sync_word` (each GPU holds its own), looked up once per device.
constexpr int kMaxDevices = 64;
int* g_sync_ptr[kMaxDevices] = {};

}  // namespace

extern "C" int tsd_accept_commit_static(const float* X_dev, const float* mu_q_dev, const float* mu_p_dev,
                                        const int32_t* round_dev, int32_t B, int32_t K, int32_t P, float sigma_p,
                                        float sigma_q, float fallback_r, uint64_t seed, uint32_t flags,
                                        int32_t* n_acc_dev, float* commit_dev, float* ell_dev, float* logu_dev,
                                        void* stream) {
  if (!X_dev || !mu_q_dev || !mu_p_dev || !n_acc_dev || !commit_dev)
    return fail_no_handle(TSD_E_INVALID_ARG, "X_dev, mu_q_dev, mu_p_dev, n_acc_dev and commit_dev must not be NULL");
  if (B < 1 || K < 1 || P < 1) return fail_no_handle(TSD_E_INVALID_ARG, "need B >= 1, K >= 1, P >= 1");
  if (B > kMaxB || K > kMaxK || (long)B * P > kMaxBP)
    return fail_no_handle(TSD_E_OUT_OF_RANGE,
                          "tsd_accept_commit_static takes at most 4096 series, K <= 16 and B * P <= 262144 "
                          "(use a handle and tsd_accept_commit beyond that)");
  if (!(sigma_p > 0.f) || !(sigma_q > 0.f) || !std::isfinite(sigma_p) || !std::isfinite(sigma_q))
    return fail_no_handle(TSD_E_INVALID_ARG, "sigma_p and sigma_q must be positive and finite");
  if (!(fallback_r >= 0.f) || fallback_r > sigma_p) return fail_no_handle(TSD_E_INVALID_ARG, "fallback_r must lie in [0, sigma_p]");
  if (flags & ~(TSD_FLAG_NO_TEMPERING | TSD_FLAG_THRESHOLD_RULE | TSD_FLAG_BATCH_SYNC | TSD_FLAG_CLEAR_REST))
    return fail_no_handle(TSD_E_INVALID_ARG,
                          "flags: only TSD_FLAG_NO_TEMPERING, TSD_FLAG_THRESHOLD_RULE, TSD_FLAG_BATCH_SYNC and TSD_FLAG_CLEAR_REST apply here");
  hipError_t e;
  hipStream_t st = (hipStream_t)stream;
  AcceptP a;
  std::memset(&a, 0, sizeof(a));
  a.X = X_dev;
  a.mu_q = mu_q_dev;
  a.mu_p = mu_p_dev;
  a.forecast = commit_dev;  // with T = K + 1 and nothing committed before, the round's patches land at [b][0 .. n]
  a.round = const_cast<int*>(round_dev);
  a.n_acc = n_acc_dev;
  a.ell = ell_dev;
  a.logu = logu_dev;
  a.B = B;
  a.K = K;
  a.P = P;
  a.T = K + 1;
  a.inv2sp2 = 1.0f / (2.0f * sigma_p * sigma_p);
  a.inv2sq2 = 1.0f / (2.0f * sigma_q * sigma_q);
  a.logdet = 0.5f * std::log((sigma_q * sigma_q) / (sigma_p * sigma_p));
  a.temper = (flags & TSD_FLAG_NO_TEMPERING) ? (float)P : 1.0f;
  a.log_alpha_override = 1.0f;
  a.fallback_r = fallback_r;
  a.key0 = (unsigned)(seed & 0xFFFFFFFFull);
  a.key1 = (unsigned)(seed >> 32);
  a.threshold = (flags & TSD_FLAG_THRESHOLD_RULE) ? 1 : 0;
  a.clear_rest = (flags & TSD_FLAG_CLEAR_REST) ? 1 : 0;
  if (flags & TSD_FLAG_BATCH_SYNC) {
    int dev = -1;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return fail_no_handle(TSD_E_HIP, std::string("hipGetDevice: ") + hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail_no_handle(TSD_E_OUT_OF_RANGE, "device index beyond 63");
    if (!g_sync_ptr[dev]) {
      // the word's name is only a host-side stand-in: the device address has to be asked for, with this device current
      int* ptr = nullptr;
      e = hipGetSymbolAddress(reinterpret_cast<void**>(&ptr), HIP_SYMBOL(sync_word));
      if (e != hipSuccess || !ptr)
        return fail_no_handle(TSD_E_HIP, std::string("hipGetSymbolAddress(sync_word): ") + hipGetErrorString(e));
      g_sync_ptr[dev] = ptr;
    }
    a.sync = g_sync_ptr[dev];
    // (a fill kernel, not a memset: the call may be captured into a graph)
    if ((e = launch_fill_int(a.sync, INT_MAX, 1, st)) != hipSuccess)
      return fail_no_handle(TSD_E_HIP, std::string("fill launch: ") + hipGetErrorString(e));
    a.mode = 1;
    if ((e = launch_accept(a, st)) != hipSuccess) return fail_no_handle(TSD_E_HIP, std::string("acceptance launch: ") + hipGetErrorString(e));
    a.mode = 2;
  }
  if ((e = launch_accept(a, st)) != hipSuccess) return fail_no_handle(TSD_E_HIP, std::string("acceptance launch: ") + hipGetErrorString(e));
  return TSD_OK;
}
