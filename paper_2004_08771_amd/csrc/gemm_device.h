// Device helpers that the dense product kernels share.
#pragma once

#include "hb_internal.h"

namespace hb {

__device__ __forceinline__ float sigmoidf_fast(float z)
{
    return __builtin_amdgcn_rcpf(1.0f + __expf(-z));  // v_rcp_f32: 1 ulp, no division sequence
}

template <int V>
struct IntC {
    static constexpr int value = V;
};
// calls f(IntC<activation>) with the run-time activation as a constant
template <typename F>
__device__ __forceinline__ void with_activation(int act, F &&f)
{
    if (act == ACT_SIGMOID) f(IntC<ACT_SIGMOID>());
    else if (act == ACT_RELU) f(IntC<ACT_RELU>());
    else f(IntC<ACT_NONE>());
}

// XCD-aware tile order: consecutive hardware workgroup ids go round-robin over the 8 XCDs,
// so give each XCD a contiguous run of the T tiles (they share an A row panel in its L2).
__device__ __forceinline__ int xcd_tile_order(int b, int T)
{
    return ((T & 7) == 0) ? (b & 7) * (T >> 3) + (b >> 3) : b;
}

}  // namespace hb
