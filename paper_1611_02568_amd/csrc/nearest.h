// Neighbour candidates (squared distance, index) and their order across a
// wavefront: nearer first, ties to the smaller index.  Distances are numbers, or
// keys that order as they do (dist_key).
#pragma once

#include "common.h"

namespace psne {
namespace {

template <typename K>
__device__ __forceinline__ bool knn_less(K da, int32_t ja, K db, int32_t jb) {
    return da < db || (da == db && ja < jb);
}

// The bits of a squared distance, which order as the distance does, with NaN after
// infinity: every pair has its place, also of rows that hold NaN.
__device__ __forceinline__ uint64_t dist_key(double d) {
    return d == d ? (uint64_t)__double_as_longlong(d) : 0x7FF8000000000000ull;
}
__device__ __forceinline__ double key_dist(uint64_t key) {
    return __longlong_as_double((long long)key);
}

// bitonic sort of one (d, j) pair per lane across the wave, ascending
template <typename K>
__device__ __forceinline__ void wave_sort(K& d, int32_t& j) {
    const int lane = lane_id();
#pragma unroll
    for (int size = 2; size <= kWave; size <<= 1) {
#pragma unroll
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const K od = __shfl_xor(d, stride, kWave);
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
