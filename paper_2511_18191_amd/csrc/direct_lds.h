// Loads from global memory straight into LDS, shared by the GEMM kernels that stage their operands this way.
#pragma once
#include <type_traits>

#include "tsd_internal.h"

namespace tsd {

#define TSD_GLOBAL_PTR(p) ((const void __attribute__((address_space(1)))*)(p))
#define TSD_LDS_PTR(p) ((void __attribute__((address_space(3)))*)(p))

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

template <int N>
struct IC : std::integral_constant<int, N> {};

// Loads J .. E - 1 of a wavefront's share of a stage: load J goes to base + J * 1024 - BIAS (the immediate must be a
// compile-time constant, hence the recursion instead of a loop; it is added to both addresses).
template <int J, int E, int BIAS>
__device__ __forceinline__ void issue_loads(const bf16* const* gp, long koff, void __attribute__((address_space(3)))* base) {
  if constexpr (J < E) {
    __builtin_amdgcn_global_load_lds(TSD_GLOBAL_PTR(gp[J] + koff), base, 16, J * 1024 - BIAS, 0);
    issue_loads<J + 1, E, BIAS>(gp, koff, base);
  }
}

}  // namespace tsd
