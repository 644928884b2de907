// Shared pieces of the matrix-core backward kernels: fragment packing from a strided (possibly transposed) source,
// the activation and its derivative, bf16 pair conversions.  See mfma.h for the operand layouts.
#pragma once
#include "gelu_grad.h"
#include "mfma.h"
#include "wavefront.h"

namespace slicemoe {

// ------------------------------------------------------------------------------------------- work split over blocks
// Rows are handed out in steps of `step` rows counted from each expert's first row, on an axis where an expert with rows
// occupies `overhead` positions, 0 or 1, more than it has steps (what it costs a block to begin an expert: its weights in, its sums out).
// Block v takes `share` consecutive positions.  A segment is what one block has of one expert; along the axis the block or
// the expert advances from one segment to the next, so v + e names a segment's slot of partial sums uniquely.
struct RowAxis {
    int first, steps;   // of lane e's expert (E <= 64): its first position, its steps
    int share;          // uniform
};
__device__ __forceinline__ RowAxis row_axis(int rows, int step, int overhead, int blocks, int lane)
{
    RowAxis A;
    A.steps = (rows + step - 1) / step;
    const int cost = A.steps > 0 ? A.steps + overhead : 0;
    A.first = wavefront_exclusive_scan(cost, lane);
    A.share = max(1, (wavefront_sum(cost) + blocks - 1) / blocks);
    return A;
}

// bf16 terms that an fp32 operand of the second-stage matrix instructions is split into.  Two (16 significant bits) where this
// backward has always run on two: 64, 96 and 128.  Three (24 bits: the operand itself) at the widths whose backward used to be
// the fp32 kernels' and stays of that precision: 24, 48 and 192.
constexpr int backward_terms(int ds) { return ds == 24 || ds == 48 || ds == 192 ? 3 : 2; }

// Weight repacking for the backward kernels: a few jobs per launch, one thread per 16-byte fragment (or bias value).
// Generic strided source so that the same code packs a matrix or its transpose: element (kk, col) of the [K, N] matrix
// being packed is src[kk * rs + col * cs] for kk < Kv and col < Nv, and zero in the padding up to K and N (multiples of
// 16 / 32).  nmat matrices, src_stride elements and dst_stride bytes apart.
//   kPackLayer1    [N/32][K/16][64]: lane (i, g), slot m: M[16ks + 8g + m][32nt + i]
//   kPackChain     [K/32][2][N/32][64]: lane (i, g), slot m: M[32ht + chain_feature(s, g, m)][32nt + i], i.e. the
//                  contraction slots follow the accumulator order; kPackChainF16: the same converted to fp16
//   kPackTile16    [K/16][N/32][64]: lane (i, g) of 16 x 4, slot m: M[16kt + i][32nt + 8g + m], the A operand of
//                  v_mfma_f32_16x16x32 (contraction over the columns)
//   kPackBias      K values per matrix widened to fp32, zero-padded to N
enum { kPackLayer1 = 0, kPackChain = 1, kPackChainF16 = 2, kPackBias = 3, kPackTile16 = 4 };
struct BwdPackJob {
    int kind, K, Kv, N, Nv;
    const bf16_t *src;
    size_t rs, cs, src_stride;
    char *dst;
    size_t dst_stride;
    long long items;   // threads this job needs
};
struct BwdPackJobs {
    int count;
    BwdPackJob job[12];
};
BwdPackJob bwd_pack_job(int kind, const void *src, int K, int Kv, int N, int Nv, size_t rs, size_t cs, size_t src_stride,
                        char *dst, size_t dst_stride, int nmat);
// In the same launch, in front: the probability sums of the capacity loss (blocks 0: none).
struct CapSums {
    int blocks;
    const int32_t *idx;
    const float *pk;
    long long Na;
    int E;
    float scale;                 // a power of two
    unsigned long long *slots;   // [blocks][E]
};
hipError_t bwd_pack_launch(const BwdPackJobs &jobs, const CapSums &cap, hipStream_t s);

// ---- The capacity loss (Section 3.2, Eq. 2) in its differentiable reading.  Eq. 2 is a function of integer counts;
// the router can only be trained with it (Section 3.1) through a stand-in, and the one taken here is the usual one: the
// count of expert e becomes the sum c_e of the final probabilities of the assignments routed to e, the loss
// alpha CV^2(c) with the population variance, and dL_cap/dp_a = alpha (2E / S^2) (c_e(a) - Q / S), S = sum c, Q = sum c^2.
// The sums are exact and the same on every run: each probability, a float in [0, 1], is added as the integer
// p * scale, 2^38 up to 2^26 assignments (capacity_scale.h; bits of a tiny p below that are rounded off).
// Bound by launches and latency, so it has no launch of its own: up to kCapBlocks blocks in front of the weight
// repacking store their sums in a slot each, and every block of the router's kernels adds the slots up for itself beside the
// staging of its weights.  Forward and backward with the two kernels for it of
// before / now: 32 208 slices at width 64 179.3 / 174.2 us; at width 96
// 11 968 slices 144.5 / 139.1, 65 528 342.9 / 342.3 (they ran beside the weight gradients).
// Large batches: what the loss adds to a backward, one assignment a load / four: width 64, 1 048 576 slices 29 / 10 us, width 24 60 / 18;
// 128 slots instead of 64 save another 5 there and cost the router's kernels 1.5 us in every batch.
constexpr int kCapBlocks = 64;
struct CapLoss {
    const unsigned long long *slots;   // null: no capacity loss
    short nslots, bits;                // bits: the sums are in units of 2^-bits
    float alpha;
};
// Thread tid of a block of WAVES wavefronts: its part of the sums into part [WAVES][64]; then, behind a barrier, the first wavefront's
// sums of those and the derivatives [64] (another barrier in front of their use).  E <= 64.
template <int WAVES>
__device__ __forceinline__ void capacity_part(const CapLoss &C, int E, int tid, unsigned long long *part)
{
    const int e = tid & 63, q = tid >> 6;
    unsigned long long sum = 0ull;
    if (e < E) {
#pragma unroll
        for (int i = 0; i < kCapBlocks / WAVES; ++i) {   // (unconditional: past the end the last slot is read and not added)
            const int b = q + i * WAVES;
            const unsigned long long v = C.slots[(size_t)min(b, C.nslots - 1) * E + e];
            sum += b < C.nslots ? v : 0ull;
        }
    }
    part[q * 64 + e] = sum;
}
template <int WAVES>
__device__ __forceinline__ void capacity_derivatives(const CapLoss &C, int E, int tid, const unsigned long long *part, float *capg)
{
    if (tid >= 64) return;
    unsigned long long sum = 0ull;
#pragma unroll
    for (int q = 0; q < WAVES; ++q) sum += part[q * 64 + tid];
    const double c = (double)sum;   // (zero for a lane without an expert)
    double S = c, Q = c * c;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        S += __shfl_xor(S, o);
        Q += __shfl_xor(Q, o);
    }
    // (S, Q and c in units of the sums: what is left of the unit goes to alpha)
    capg[tid] = S > 0.0 ? (float)(ldexp((double)C.alpha, C.bits) * (2.0 * E / (S * S)) * (c - Q / S)) : 0.f;
}

// Append what the expert part and the router part need (three or four jobs, and seven); `packed` and `scratch` are their regions.
void backward_expert_pack_jobs(const slicemoe_config &c, const BackwardWeightsPlan &W, const slicemoe_weights &w, void *packed, BwdPackJobs &jobs);
void backward_router_pack_jobs(const slicemoe_config &c, const slicemoe_weights &w, void *scratch, BwdPackJobs &jobs);

// Backward copies of one expert's weights in fragment order (bytes from the start of the expert's block).
//   w1f  [HT][KS][64]      W1 fragments as the forward packs them: lane (i, g), slot m: W1[16ks + 8g + m][32ht + i]
//   w2r  [HT][KS][64]      rows of W2: lane (i, g), slot m: W2[32ht + i][16ks + 8g + m]
//   w1c  [HT][2][OT][64]   W1 with the hidden units as contraction slots in accumulator order:
//                          lane (i, g), slot m: W1[32ot + i][32ht + chain_feature(s, g, m)]
//   w1d  [FT][HT][64]      the same for 16-feature tiles: lane (i, g) of 16 x 4, slot m: W1[16ft + i][32ht + 8g + m]
//                          (one of w1c and w1d is there: w1d when the fused kernel runs; neither where only the one-pass kernel does)
//   b1   [He] fp32
struct BwdPacked {
    size_t w1f, w2r, w1c, w1d, b1, stride;
};
// Matrix-core expert weight gradients (backward_weights_mfma.hip): the split of the rows and the launches.  fused: the
// kernel also writes dL/dx and dL/dp of the rows.
struct BackwardWeightsPlan {
    bool onepass, fused;   // onepass: bwd_expert_kernel (then fused too)
    int step, groups, blocks;
    int overhead;          // of an expert, on the axis of the work split: 0 or 1
    // Slots of partial weight gradients: those that this batch uses, and those to reserve -- at least as many, and never fewer for more
    // tokens, so that a workspace made for a layer's largest batch takes its smaller ones, whichever kernels those run on.
    long long slots, reserve;
};
constexpr bool weights_fused(int ds, int He) { return ds == 64 && He <= 256; }
BackwardWeightsPlan backward_weights_plan(const slicemoe_config &c);
BackwardWeightsPlan backward_expert_plan(const slicemoe_config &c);   // of the one-pass kernel (backward_expert_mfma.hip)
hipError_t launch_backward_expert_onepass(const slicemoe_config &c, const BackwardWeightsPlan &W, const BwdPacked &L, const void *h, const void *d_out,
                                          const float *pk, const int32_t *offsets, const int32_t *perm, const char *packed, size_t slot_floats,
                                          float *part, float *dxrow, float *dpk, hipStream_t s);
BackwardWeightsPlan backward_generic_plan(const slicemoe_config &c);   // of the fp32 expert kernel (backward_generic.hip)
hipError_t launch_backward_weights(const slicemoe_config &c, const BackwardWeightsPlan &W, const BwdPacked &L, const void *h, const void *d_out, const float *pk,
                                   const int32_t *offsets, const int32_t *perm, const char *packed, size_t slot_floats, float *part,
                                   float *dxrow, float *dpk, hipStream_t s);

// Twice GELU and twice its derivative of four values (the factors of two, exact, are taken out of the finished sums).  With x = |z|,
// e = exp(-x^2 / 2), t = 1 / (1 + 0.3 x) and the quintic N(t) of gelu_grad.h: q = 2 Phi(-x) = e - x e N, 2 z Phi(z) = (z + x) - x q, and with
// p = 2 Phi(z), which is q below zero and 2 - q above, twice the derivative is p + 2 z phi(z).  q keeps a precision of its own, where
// z (1 + erf) below zero has that of one.  Relative 2-norm of the error against 64-bit arithmetic, activation / derivative
// (fp32, half a unit of error in the hardware's exponential):
//                        this                                  1 + erf, same N          erff and expf            A & S 7.1.26
//   z ~ N(0, 0.1 .. 2.5) 2.4e-8 .. 4.7e-8 / 4.0e-8 .. 5.5e-8   2.9e-8 .. 4.4e-8 / 4.9e-8   3.3e-8 .. 4.0e-8 / 4.0e-8  5.9e-8 .. 1.5e-7 / 1.7e-7
//   z ~ N(-2, 0.3)       1.8e-7 / 1.3e-7                       4.9e-7 / 2.7e-7          3.3e-7 / 1.3e-7          1.7e-6 / 6.7e-7
//   z ~ N(-5, 0.3)       5.4e-5 / 2.9e-6                       6.7e-3 / 5.5e-4          4.7e-3 / 2.2e-4          7.3e-4 / 3.9e-5
// The step from q to 2 - q is a product with infinity, clamped to 0 .. 1 (no number for z = 0, which the clamp makes 0: p = 1 either way): a comparison and a
// selection write and wait for a mask (backward of 32 768 tokens at width 96 660 us with them, 650 without; width 128 2377, 2349).
// Four side by side: a vector instruction that needs the result of the one before waits 8.3 cycles for it.
__device__ __forceinline__ void twice_gelu4(const float (&z)[4], float (&act)[4], float (&slope)[4])
{
    float e[4], t[4], n[4], q[4], ze[4], above[4];
#define SLICEMOE_EACH for (int i = 0; i < 4; ++i)
#pragma unroll
    SLICEMOE_EACH t[i] = fmaf(kGeluGradP, fabsf(z[i]), 1.f);
#pragma unroll
    SLICEMOE_EACH e[i] = z[i] * -0.72134752044448170f;   // exp(-z^2 / 2) = 2^(-z^2 log2(e) / 2)
#pragma unroll
    SLICEMOE_EACH t[i] = __builtin_amdgcn_rcpf(t[i]);
#pragma unroll
    SLICEMOE_EACH e[i] = __builtin_amdgcn_exp2f(e[i] * z[i]);
#pragma unroll
    SLICEMOE_EACH n[i] = fmaf(kGeluGradN[0], t[i], kGeluGradN[1]);
#pragma unroll
    for (int c = 2; c < 6; ++c)
#pragma unroll
        SLICEMOE_EACH n[i] = fmaf(n[i], t[i], kGeluGradN[c]);
#pragma unroll
    SLICEMOE_EACH ze[i] = e[i] * z[i];
#pragma unroll
    SLICEMOE_EACH above[i] = __builtin_amdgcn_fmed3f(z[i] * __builtin_inff(), 0.f, 1.f);   // 1 above zero, 0 below
#pragma unroll
    SLICEMOE_EACH q[i] = fmaf(-fabsf(ze[i]), n[i], e[i]);
#pragma unroll
    SLICEMOE_EACH act[i] = z[i] + fabsf(z[i]);
#pragma unroll
    SLICEMOE_EACH act[i] = fmaf(-fabsf(z[i]), q[i], act[i]);
#pragma unroll
    SLICEMOE_EACH q[i] = fabsf(fmaf(2.f, above[i], -q[i]));   // p
#pragma unroll
    SLICEMOE_EACH slope[i] = fmaf(0.79788456080286536f, ze[i], q[i]);
#undef SLICEMOE_EACH
}

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b)   // round to nearest even
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    const f32x2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// TERMS-term bf16 split of four values, the largest term first: 8 significant bits each.
template <int TERMS>
__device__ __forceinline__ void split_terms(const float (&v)[4], uint32_t (&out)[TERMS][4], int i)
{
    float r[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
    for (int t = 0; t < TERMS; ++t) {
        const uint32_t h0 = pack_bf16x2(r[0], r[1]), h1 = pack_bf16x2(r[2], r[3]);
        out[t][i] = h0;
        out[t][i + 1] = h1;
        if (t + 1 < TERMS) {
            r[0] -= __uint_as_float(h0 << 16);
            r[1] -= __uint_as_float(h0 & 0xffff0000u);
            r[2] -= __uint_as_float(h1 << 16);
            r[3] -= __uint_as_float(h1 & 0xffff0000u);
        }
    }
}

__device__ __forceinline__ bf16x8 frag_of(const uint32_t (&p)[8], int s)   // K-step s of eight register pairs
{
    return __builtin_bit_cast(bf16x8, make_uint4(p[4 * s], p[4 * s + 1], p[4 * s + 2], p[4 * s + 3]));
}

// Block-wide copy of `bytes` (a multiple of 16) from memory to LDS; callers synchronise.
__device__ __forceinline__ void stage_bytes(const char *__restrict__ src, char *lds, size_t bytes, int tid, int nthreads)
{
    const uint4 *g = (const uint4 *)src;
    uint4 *l = (uint4 *)lds;
    const int n = (int)(bytes / 16);
    for (int i = tid; i < n; i += nthreads) l[i] = g[i];
}

}  // namespace slicemoe
