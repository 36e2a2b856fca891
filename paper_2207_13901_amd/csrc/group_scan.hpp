// Sums of counts over the lanes of a workgroup.
#pragma once

#include <cstdint>

namespace spl {

// Inclusive sum over the T lanes (whole waves of 64) of the workgroup; *all
// gets the total.  In 64 bits: a row's count of entries fits 32, the sum over
// a few dozen long rows need not.  s_wave: T / 64 entries of LDS.
template <int T>
__device__ __forceinline__ int64_t group_inclusive(int64_t v, int64_t *s_wave, int64_t *all) {
    constexpr int kLanes = 64;
    const int lane = threadIdx.x % kLanes, wave = threadIdx.x / kLanes;
#pragma unroll
    for (int off = 1; off < kLanes; off <<= 1) {
        const int64_t u = __shfl_up(v, off);
        v += lane >= off ? u : 0;
    }
    if (lane == kLanes - 1) s_wave[wave] = v;
    __syncthreads();
    int64_t total = 0;
#pragma unroll
    for (int w = 0; w < T / kLanes; ++w) {
        v += w < wave ? s_wave[w] : 0;
        total += s_wave[w];
    }
    *all = total;
    return v;
}

}  // namespace spl
