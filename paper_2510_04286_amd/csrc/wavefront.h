// Sums and prefix sums over the lanes of a wavefront, without the LDS.
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

// Sums over the 32 lanes of a lane group of 16 values each, half of the values at every exchange, so that what is left
// spreads over the lanes: 32 instructions.  Afterwards v[0] and v[1] are the sums of the values that were registers
// acc-order rows hidden_sum_row(lane) and + 1 (the four lanes of a quad hold the same).  The additions of a lane's own
// value and one from another lane of its row of 16 are single instructions whose bank mask restricts them to the lanes
// (banks of four) that keep that value; each group starts with the two wait states a moved operand needs.
__device__ __forceinline__ float sum_over_row_pair(float a, float b)   // even rows of 16 lanes keep a, odd ones b
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ void sum_over_hidden(float (&v)[8])   // v[i]: sum_over_row_pair of values i and i + 8
{
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %2, %2, %2 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %3, %3, %3 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %0, %4, %4 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %1, %5, %5 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %2, %6, %6 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %3, %7, %7 row_ror:8 row_mask:0xf bank_mask:0xc"
        : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3])
        : "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]));
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %0, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %1, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xa"
        : "+v"(v[0]), "+v"(v[1])
        : "v"(v[2]), "v"(v[3]));
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        v[i] += __int_as_float(lane_move<0xB1>(__float_as_int(v[i])));   // quad_perm [1, 0, 3, 2]
        v[i] += __int_as_float(lane_move<0x4E>(__float_as_int(v[i])));   // quad_perm [2, 3, 0, 1]
    }
}
__device__ __forceinline__ int hidden_sum_row(int lane)
{
    return 16 * ((lane >> 4) & 1) + 8 * ((lane >> 3) & 1) + 4 * (lane >> 5) + 2 * ((lane >> 2) & 1);
}

// Orders LDS traffic between the lanes of one wavefront (the hardware keeps a wavefront's LDS operations in order; this
// keeps the compiler from moving them across).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace slicemoe
