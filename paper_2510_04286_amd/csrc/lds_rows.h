// Rows of bf16 values in the LDS, read both ways by the matrix-core backward kernels: as they are (a lane per row) and
// transposed (a lane per column, by ds_read_b64_tr_b16).
#pragma once
#include "mfma.h"

namespace slicemoe {

typedef short s16x4 __attribute__((ext_vector_type(4)));

// PW 16-byte pieces per row (a power of two; the pieces past the slice width stay zero), the piece index XORed with a
// function of the row so that both ways of reading are free of bank conflicts: as A operand (32 lanes, one row each, the
// same piece) and transposed (4 rows x 64 bytes per half-wavefront).
template <int DS> struct LdsRows {
    static constexpr int P = DS / 8;
    static constexpr int PW = P <= 4 ? 4 : P <= 8 ? 8 : P <= 16 ? 16 : P <= 32 ? 32 : 64;
    static constexpr int STRIDE = PW * 16;
    static __device__ __forceinline__ int swizzle(int row)
    {
        return PW == 4 ? (row >> 2) & 3 : PW == 8 ? (((row >> 1) & 1) << 2) | ((row >> 2) & 3) : ((row & 3) << 2) | ((row >> 2) & 3);
    }
    static __device__ __forceinline__ int offset(int row, int piece) { return row * STRIDE + ((piece ^ swizzle(row)) << 4); }
};

typedef __attribute__((address_space(3))) char *lds_ptr;
__device__ __forceinline__ lds_ptr as_lds(const char *p) { return (lds_ptr)p; }

// a / k for assignment ids (0 <= a < 2^31) and 1 <= k <= 8, uniform k: a shift, or one high multiplication (with
// m = ceil(2^(32 + s) / k) the excess e = m k - 2^(32 + s) < k keeps a e below 2^(32 + s)).
__device__ __forceinline__ int divide_by_k(int a, int k)
{
    if ((k & (k - 1)) == 0) return a >> (31 - __clz(k));
    const unsigned m = k == 3 ? 2863311531u : k == 5 ? 3435973837u : k == 6 ? 2863311531u : 2454267027u;
    return (int)(__umulhi((unsigned)a, m) >> (k == 3 ? 1 : 2));
}

// Two transposing reads: slots 0..3 from the four rows at `a`, slots 4..7 from those at `b`.
__device__ __forceinline__ bf16x8 read_transposed(lds_ptr a, lds_ptr b)
{
    union {
        s16x4 h[2];
        bf16x8 v;
    } r;
    r.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)a);
    r.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)b);
    return r.v;
}

// Sum of the eight bf16 values of a fragment.
__device__ __forceinline__ float fragment_sum(bf16x8 f)
{
    const uint4 u = __builtin_bit_cast(uint4, f);
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) s += __uint_as_float(w[i] << 16) + __uint_as_float(w[i] & 0xffff0000u);
    return s;
}

}  // namespace slicemoe
