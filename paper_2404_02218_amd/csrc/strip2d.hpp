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

// entries of a row-sorted list [from, end) above row y, counted by the wave
__device__ __forceinline__ int rows_before(const int* zyx4, int from, int end, int y) {
    int n = 0;
    for (int e0 = from; e0 < end; e0 += 64) {
        const int e = e0 + ((int)threadIdx.x & 63);
        n += __popcll(__ballot(e < end && zyx4[4 * e + 1] < y));
    }
    return n;
}

}  // namespace stn
