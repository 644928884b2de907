// Sums and prefix sums over the 64 lanes of a wavefront, without the LDS.
#pragma once
#include <hip/hip_runtime.h>

namespace slicemoe {

template <int CTRL> __device__ __forceinline__ int lane_move(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true); }

__device__ __forceinline__ int wavefront_sum(int v)
{
    v += lane_move<0xB1>(v);    // quad_perm [1, 0, 3, 2]
    v += lane_move<0x4E>(v);    // quad_perm [2, 3, 0, 1]
    v += lane_move<0x141>(v);   // row_half_mirror
    v += lane_move<0x140>(v);   // row_mirror: every lane now holds the sum of its row of 16
    return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) +
           __builtin_amdgcn_readlane(v, 48);
}

__device__ __forceinline__ int wavefront_exclusive_scan(int v, int lane)
{
    int s = v;
    s += lane_move<0x111>(s);   // row_shr 1, 2, 4, 8 with zero fill: inclusive scan inside a row of 16
    s += lane_move<0x112>(s);
    s += lane_move<0x114>(s);
    s += lane_move<0x118>(s);
    const int r0 = __builtin_amdgcn_readlane(s, 15), r1 = __builtin_amdgcn_readlane(s, 31), r2 = __builtin_amdgcn_readlane(s, 47);
    const int row = lane >> 4;
    return s - v + (row == 0 ? 0 : row == 1 ? r0 : row == 2 ? r0 + r1 : r0 + r1 + r2);
}

}  // namespace slicemoe
