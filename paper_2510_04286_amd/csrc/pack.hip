// One-time re-tiling of the bf16 weights into matrix-core fragment order (see mfma.h for the
// operand layout).  A fragment is the 16 bytes one lane feeds to one MFMA: 8 bf16 along the
// contraction dimension.  Biases are widened to fp32.  One thread per fragment / bias element.
//
// Router   W1 frags [Hr/32][ds/16][64 lanes]      lane (i, g), slot m: Wr1[16*ks + 8*g + m][32*ht + i]
//          (ds/16 and ds/32 rounded up: rows and columns past ds are zeros)
//          W2 frags [Epad/32][Hr/32][2][64]       lane (i, g), slot m: Wr2[32*ht + chain_feature(s,g,m)][32*et + i], as fp16
// Expert e W1 frags [He/32][ds/16][64]            kappa * W1[e][16*ks + 8*g + m][32*ht + i]   (kappa = 1/4: exact in bf16)
//          W2 frags [He/32][2][ds/32][64]         W2[e][32*ht + chain_feature(s,g,m)][32*ot + i] / kappa, as fp16
//          b1       [He/32][2 lane groups][16]    kappa * b1[e][32*ht + acc_feature(r, g)], as fp16
//          b2       [ds rounded up to 32] fp32
// The expert kernel evaluates its activation on s = kappa z in packed fp16 (see ffn_mfma.hip), so
// its second GEMM runs on fp16 fragments; bf16 weights convert exactly to fp16 unless they are
// smaller than 2^-14 / 4 (rounded, absolute error below 2^-27) or beyond +-16376 (clamped).
#include "mfma.h"

namespace slicemoe {

__device__ __forceinline__ void store_frag(char *dst, const bf16_t v[8])
{
    uint4 u;
    u.x = v[0] | ((uint32_t)v[1] << 16);
    u.y = v[2] | ((uint32_t)v[3] << 16);
    u.z = v[4] | ((uint32_t)v[5] << 16);
    u.w = v[6] | ((uint32_t)v[7] << 16);
    *(uint4 *)dst = u;
}

// The eight pieces of the packed buffer as jobs of one launch: fragments of 16 bytes or single bias values, numbered one
// job after the other, one thread each.  One launch because the pieces are small (128 KiB to 8 MiB): eight launches in a
// stream cost 4.5-6 us each, whatever they move; together a training step became 31 us shorter (T = 16384, d = 1024,
// S = 16, E = 32: 804 -> 773 us; d = 768, S = 8, T = 8191: 485 -> 458 us).
//   kLayer1   first-layer matrix W[K, N] (row-major), A operand of the transposed GEMM1, times `scale` (a power of
//             two: the product is again a bf16 value, exactly, unless it falls into the subnormal range below 2^-126);
//             rows K..Kpad-1 are zeros
//   kLayer2   second-layer matrix W[K, N] as fp16 times `scale`, A operand of the transposed GEMM2 whose contraction slots
//             follow the accumulator layout of GEMM1; columns N..Npad-1 are zeros.  outer_first lays the fragments out as
//             [nt][ht][s][lane] (router), otherwise as [ht][s][nt][lane] (experts)
//   kBiasF16  N biases as fp16, times `scale`, in the accumulator order of each hidden tile
//   kBias     N biases widened to fp32, zero-padded to Npad
enum { kLayer1, kLayer2, kBiasF16, kBias };
struct PackJob {
    int kind, K, Kpad, N, Npad, outer_first;
    float scale;
    unsigned per;            // items per matrix
    unsigned items;          // items of all matrices
    size_t src_stride;       // elements between matrices
    const bf16_t *src;
    char *dst;
    size_t dst_stride;       // bytes between matrices
};
constexpr int kPackJobs = 8;
struct PackJobs {
    PackJob job[kPackJobs];
};

__device__ __forceinline__ bf16_t clamped_f16(bf16_t w, float scale)
{
    const _Float16 hv = (_Float16)fminf(fmaxf(bf16_to_f32(w) * scale, -65504.f), 65504.f);
    return __builtin_bit_cast(bf16_t, hv);
}

__device__ __forceinline__ void pack_item(const PackJob &J, unsigned f)
{
    const unsigned mat = f / J.per, item = f - mat * J.per;
    const bf16_t *src = J.src + (size_t)mat * J.src_stride;
    char *dst = J.dst + (size_t)mat * J.dst_stride;
    if (J.kind == kBias) {
        ((float *)dst)[item] = (int)item < J.N ? bf16_to_f32(src[item]) : 0.f;
        return;
    }
    if (J.kind == kBiasF16) {
        const int ht = (int)item / 32, g = ((int)item % 32) / 16, r = (int)item % 16;
        ((bf16_t *)dst)[item] = clamped_f16(src[32 * ht + acc_feature(r, g)], J.scale);
        return;
    }
    const int lane = (int)(item % 64), i = lane & 31, g = lane >> 5;
    int r = (int)(item / 64);
    bf16_t v[8];
    if (J.kind == kLayer1) {
        const int KS = J.Kpad / 16, ks = r % KS, ht = r / KS;
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int kk = 16 * ks + 8 * g + m;
            v[m] = kk < J.K ? f32_to_bf16(bf16_to_f32(src[(size_t)kk * J.N + 32 * ht + i]) * J.scale) : (bf16_t)0;
        }
    } else {
        const int HT = J.K / 32, NT = J.Npad / 32;
        int ht, s, nt;
        if (J.outer_first) {
            s = r % 2;
            r /= 2;
            ht = r % HT;
            nt = r / HT;
        } else {
            nt = r % NT;
            r /= NT;
            s = r % 2;
            ht = r / 2;
        }
        const int col = 32 * nt + i;
#pragma unroll
        for (int m = 0; m < 8; ++m)
            v[m] = clamped_f16(col < J.N ? src[(size_t)(32 * ht + chain_feature(s, g, m)) * J.N + col] : (bf16_t)0, J.scale);
    }
    store_frag(dst + (size_t)item * 16, v);
}

__global__ __launch_bounds__(256) void pack_kernel(PackJobs jobs)
{
    unsigned f = blockIdx.x * 256u + threadIdx.x;
#pragma unroll
    for (int q = 0; q < kPackJobs; ++q) {
        if (f < jobs.job[q].items) {
            pack_item(jobs.job[q], f);
            return;
        }
        f -= jobs.job[q].items;
    }
}

static PackJob pack_job(int kind, const void *src, int K, int Kpad, int N, int Npad, int outer_first, float scale, size_t src_stride,
                        char *dst, size_t dst_stride, int nmat)
{
    PackJob J;
    J.kind = kind;
    J.K = K; J.Kpad = Kpad; J.N = N; J.Npad = Npad;
    J.outer_first = outer_first;
    J.scale = scale;
    J.per = kind == kLayer1 ? (unsigned)(N / 32 * (Kpad / 16) * 64) : kind == kLayer2 ? (unsigned)(K / 32 * 2 * (Npad / 32) * 64)
          : (unsigned)Npad;
    J.items = J.per * (unsigned)nmat;
    J.src_stride = src_stride;
    J.src = (const bf16_t *)src;
    J.dst = dst;
    J.dst_stride = dst_stride;
    return J;
}

hipError_t launch_pack(const slicemoe_config &c, const slicemoe_weights &w, void *packed, hipStream_t s)
{
    const PackedLayout L = packed_layout(c);
    char *base = (char *)packed, *eb = base + L.experts;
    const int ds = L.ds, Hr = L.Hr, He = L.He, E = L.E;
    // items are counted in 32 bits, as threads of a launch are: a launch per piece where all pieces together exceed that
    const unsigned long long most = 0xffffff00ull, frags = (unsigned long long)E * (L.dsK > L.dsN ? L.dsK : L.dsN) * He / 8;
    if (frags > most) return hipErrorInvalidValue;
    PackJobs P;
    P.job[0] = pack_job(kLayer1, w.W1, ds, L.dsK, He, He, 0, kGeluKappa, (size_t)ds * He, eb + L.e_w1, L.e_stride, E);
    P.job[1] = pack_job(kLayer2, w.W2, He, He, ds, L.dsN, 0, 1.f / kGeluKappa, (size_t)He * ds, eb + L.e_w2, L.e_stride, E);
    P.job[2] = pack_job(kBiasF16, w.b1, 1, 1, He, He, 0, kGeluKappa, (size_t)He, eb + L.e_b1, L.e_stride, E);
    P.job[3] = pack_job(kBias, w.b2, 1, 1, ds, L.dsN, 0, 1.f, (size_t)ds, eb + L.e_b2, L.e_stride, E);
    P.job[4] = pack_job(kLayer1, w.Wr1, ds, L.dsK, Hr, Hr, 0, 1.f, 0, base + L.r_w1, 0, 1);
    P.job[5] = pack_job(kLayer2, w.Wr2, Hr, Hr, E, L.Epad, 1, 1.f, 0, base + L.r_w2, 0, 1);
    P.job[6] = pack_job(kBias, w.br1, 1, 1, Hr, Hr, 0, 1.f, 0, base + L.r_b1, 0, 1);
    P.job[7] = pack_job(kBias, w.br2, 1, 1, E, L.Epad, 0, 1.f, 0, base + L.r_b2, 0, 1);
    unsigned long long total = 0;
    for (const PackJob &J : P.job) total += J.items;
    if (total <= most) {
        pack_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>(P);
        return hipGetLastError();
    }
    for (int q = 0; q < kPackJobs; ++q) {
        PackJobs one = P;
        for (int r = 0; r < kPackJobs; ++r)
            if (r != q) one.job[r].items = 0;
        pack_kernel<<<(P.job[q].items + 255) / 256, 256, 0, s>>>(one);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace slicemoe
