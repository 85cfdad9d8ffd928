// Shared by the 2D sweeps by strips (step2d.hip, march2d.hip): a wavefront owns
// 256 consecutive x points of a row, 4 per lane.
#pragma once

#include "zmarch.hpp"

namespace stn {

// the neighbouring lane's value (0 past the ends of the wave, where it only
// feeds points that the neighbouring strip owns)
__device__ __forceinline__ float from_left(float x) {    // lane - 1
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_right(float x) {   // lane + 1
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130, 0xf, 0xf, true));
}

// order LDS accesses of the lanes of one wave (they run in program order)
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Searches of a sorted list's range [from, end) by the whole wave for the first
// entry that does not lie before (z, y): lists by strip are sorted by y (z is 0
// there), lists by tile by z and then y.  64 entries evenly apart narrow the
// range 64 times a round.
__device__ __forceinline__ int entries_before(const int* zyx4, int e, int end, int z, int y) {
    const int4 q = reinterpret_cast<const int4*>(zyx4)[min(e, end - 1)];
    return __popcll(__ballot(e < end && (q.x < z || (q.x == z && q.y < y))));
}
// an entry at or less than 64 in front of it (no load for up to 64 entries)
__device__ __forceinline__ int near_first(const int* zyx4, int from, int& end, int z, int y) {
    while (end - from > 64) {
        const int step = (end - from + 63) >> 6;
        const int n = entries_before(zyx4, from + ((int)threadIdx.x & 63) * step, end, z, y);
        if (n == 0) {
            end = from;
        } else {
            end = min(end, from + n * step);
            from += (n - 1) * step + 1;
        }
    }
    return from;
}
// the entry itself, or `end`
__device__ __forceinline__ int first_from(const int* zyx4, int from, int end, int z, int y) {
    from = near_first(zyx4, from, end, z, y);
    return from < end ? from + entries_before(zyx4, from + ((int)threadIdx.x & 63), end, z, y) : from;
}

}  // namespace stn
