// Mean of fp32 partial sums by one workgroup, in a fixed order.
#pragma once
#include "common.hpp"

namespace mp {

constexpr int MEAN_THREADS = 256;
constexpr int MEAN_LOADS   = 16;  // partials a thread has on their way, where there are that many

// Bound by memory latency: a thread has 16 loads on their way at a time and adds them in index order, so 8192 row losses
// cost two round trips and not 32 (8192 x 32768 vocabulary iteration 1840 -> 1834 us; the kernel took 12.7 us before).
// LOADS 1 is for up to one partial per thread, where 16 loads each cost 0.2 us more than one (losses of 1 to 100 rows).
template <int LOADS>
__device__ __forceinline__ void mean_of_parts(const float* __restrict__ part, const int n, const double denom, float* __restrict__ out) {
    __shared__ float red[MEAN_THREADS / 64];
    float            acc = 0.f;
    for (long long i = threadIdx.x; i < n; i += LOADS * MEAN_THREADS) {
        float v[LOADS];
#pragma unroll
        for (int k = 0; k < LOADS; ++k) v[k] = part[min(i + k * MEAN_THREADS, (long long)n - 1)];
#pragma unroll
        for (int k = 0; k < LOADS; ++k) acc += i + k * MEAN_THREADS < n ? v[k] : 0.f;
    }
    const float tot = block_sum<MEAN_THREADS / 64>(acc, red);
    if (threadIdx.x == 0) *out = tot / (float)denom;
}

}  // namespace mp
