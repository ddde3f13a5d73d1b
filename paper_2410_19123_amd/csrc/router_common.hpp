// Shared by the router block's kernels (router_tf.hip, router_fused.hip).
#pragma once

#include "common.hpp"
#include "internal.hpp"

namespace readme {

// Request offsets staged in LDS for the position search when they fit.
constexpr int kRoLds = 4096;

// Position of token t in its request: t - ro[r] for the last r with
// ro[r] <= t (ro = request offsets [R + 1], ro[0] = 0, ro[R] = T).
__device__ __forceinline__ int32_t position_of(int64_t t, int32_t R,
                                               const int32_t* __restrict__ ro) {
    int lo = 0, hi = R;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (ro[mid] <= t) lo = mid;
        else hi = mid;
    }
    int64_t start = ro[lo];
    if (start < 0) start = 0;
    if (start > t) start = t;
    return (int32_t)(t - start);
}

// Sum over the wave to lane 0 in a fixed order, then broadcast, so that every
// lane holds the same fp32 total.
__device__ __forceinline__ float wave_sum_bcast(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_down(v, off, 64);
    return __shfl(v, 0, 64);
}

}  // namespace readme
