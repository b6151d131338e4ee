// Neighbour candidates (squared distance, index) and their order across a
// wavefront: nearer first, ties to the smaller index.
#pragma once

#include "common.h"

namespace psne {
namespace {

__device__ __forceinline__ bool knn_less(double da, int32_t ja, double db, int32_t jb) {
    return da < db || (da == db && ja < jb);
}

// bitonic sort of one (d, j) pair per lane across the wave, ascending
__device__ __forceinline__ void wave_sort(double& d, int32_t& j) {
    const int lane = lane_id();
#pragma unroll
    for (int size = 2; size <= kWave; size <<= 1) {
#pragma unroll
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const double od = __shfl_xor(d, stride, kWave);
            const int32_t oj = __shfl_xor(j, stride, kWave);
            const bool up = (lane & size) == 0;          // this block sorts ascending
            const bool low = (lane & stride) == 0;       // this lane holds the lower slot
            const bool other_less = knn_less(od, oj, d, j);
            // the lower slot of an ascending block keeps the smaller pair
            const bool take = (low == up) ? other_less : knn_less(d, j, od, oj);
            if (take) {
                d = od;
                j = oj;
            }
        }
    }
}

}  // namespace
}  // namespace psne
