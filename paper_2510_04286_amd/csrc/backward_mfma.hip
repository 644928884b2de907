// Matrix-core backward of the expert stage: the recomputed pre-activations, dL/dz, dL/dx, dL/dp and the expert weight
// gradients of the backward pass described in backward.hip, on v_mfma_f32_32x32x16_bf16, for the slice widths the forward's
// matrix-core kernels have except 384, and any hidden width that is a multiple of 32.
//
//   bwd_rows_streamed_mfma_kernel   (here) the forward's layout: a lane owns one stacked row (see mfma.h).  Per 32-row
//                            unit and 32-wide hidden tile: u = W1^T x and da = W2 dy (weight fragment = A operand, row
//                            fragment = B), then per lane z = p u + b1, dz = da gelu'(z), and dx += W1 (p dz) with
//                            p dz fed from the accumulator registers as the B operand, exactly like the forward's
//                            second GEMM.  dL/dp = sum over the hidden units of dz u is a per-lane sum plus one
//                            exchange with lane ^ 32.  Writes dL/dx of the rows (fp32) and dL/dp.
//   bwd_weights_kernel       (backward_weights_mfma.hip) the transposed layout, for the weight gradients; at width 64, for experts
//                            whose hidden tiles fit one block, it gives dL/dx and dL/dp too, and this kernel does not run.
//   bwd_expert_kernel        (backward_expert_mfma.hip) all of it in one pass, 16 hidden units per wavefront: widths 24, 48, 96.
//
// Precision: u, da, z, the activation and its derivative in fp32 (twice_gelu4); the operands of the
// second-stage matrix instructions (p dz, a1) enter as two-term bf16 splits (hi + lo, 16 significant bits, one
// matrix instruction per term against exact bf16 data), so the results are of fp32 grade; three terms (24 significant
// bits) at widths 24, 48 and 192 (backward_terms), which are as close to 64-bit arithmetic as the fp32 kernels.  The kernels are
// bound by vector instructions, not by the matrix pipe, so a further term costs little.
#include "bwd_mfma.h"
#include "onepass_split.h"

namespace slicemoe {

static BwdPacked bwd_packed_layout(const slicemoe_config &c)
{
    BwdPacked L;
    const int ds = c.d / c.S, He = c.He;
    // (w1c has its place for every batch of a layer if it has for some: the size never falls as the batch grows)
    const bool onepass = onepass_in_every_batch(ds, He), fused = weights_fused(ds, He);
    const size_t dsK = (size_t)(ds + 15) / 16 * 16, dsN = (size_t)(ds + 31) / 32 * 32;
    L.w1f = 0;
    L.w2r = dsK * He * 2;
    L.w1c = L.w1d = 2 * L.w2r;
    L.b1 = L.w1c + (onepass ? 0 : fused ? dsK : dsN) * He * 2;
    L.stride = align_up(L.b1 + (size_t)He * 4, 256);
    return L;
}

// One thread per fragment (or bias value) of one job; see bwd_mfma.h for the layouts.
__device__ __forceinline__ void pack_layer1_item(const BwdPackJob &J, long long f)
{
    const int KS = J.K / 16;
    const long long per = (long long)(J.N / 32) * KS * 64;
    const int mat = (int)(f / per);
    long long r = f - (long long)mat * per;
    const int lane = (int)(r % 64);
    r /= 64;
    const int ks = (int)(r % KS), nt = (int)(r / KS);
    const int i = lane & 31, g = lane >> 5;
    const bf16_t *src = J.src + (size_t)mat * J.src_stride;
    const int col = 32 * nt + i;
    uint32_t v[4];
    if (J.rs == 1 && J.Kv == J.K && J.cs % 8 == 0 && col < J.Nv && ((uintptr_t)src & 15) == 0) {   // eight consecutive values
        *(uint4 *)(J.dst + (size_t)mat * J.dst_stride + (size_t)(f - (long long)mat * per) * 16) =
            *(const uint4 *)(src + (size_t)col * J.cs + 16 * ks + 8 * g);
        return;
    }
    for (int m = 0; m < 8; m += 2) {
        const int k0 = 16 * ks + 8 * g + m;
        const uint32_t lo = (k0 < J.Kv && col < J.Nv) ? src[(size_t)k0 * J.rs + (size_t)col * J.cs] : 0;
        const uint32_t hi = (k0 + 1 < J.Kv && col < J.Nv) ? src[(size_t)(k0 + 1) * J.rs + (size_t)col * J.cs] : 0;
        v[m / 2] = lo | (hi << 16);
    }
    *(uint4 *)(J.dst + (size_t)mat * J.dst_stride + (size_t)(f - (long long)mat * per) * 16) = make_uint4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ void pack_chain_item(const BwdPackJob &J, long long f)
{
    const int HT = J.K / 32, NT = J.N / 32;
    const long long per = (long long)HT * 2 * NT * 64;
    const int mat = (int)(f / per);
    long long r = f - (long long)mat * per;
    const int lane = (int)(r % 64);
    r /= 64;
    const int nt = (int)(r % NT);
    r /= NT;
    const int s = (int)(r % 2), ht = (int)(r / 2);
    const int i = lane & 31, g = lane >> 5;
    const bf16_t *src = J.src + (size_t)mat * J.src_stride;
    const int col = 32 * nt + i;
    uint32_t v[4];
    for (int m = 0; m < 8; m += 2) {
        uint32_t pr[2];
        for (int c = 0; c < 2; ++c) {
            const int kk = 32 * ht + chain_feature(s, g, m + c);
            bf16_t w = (kk < J.Kv && col < J.Nv) ? src[(size_t)kk * J.rs + (size_t)col * J.cs] : (bf16_t)0;
            if (J.kind == kPackChainF16) {   // bf16 values convert exactly unless tiny (rounded) or beyond the fp16 range (clamped)
                const _Float16 hv = (_Float16)fminf(fmaxf(bf16_to_f32(w), -65504.f), 65504.f);
                w = __builtin_bit_cast(bf16_t, hv);
            }
            pr[c] = w;
        }
        v[m / 2] = pr[0] | (pr[1] << 16);
    }
    *(uint4 *)(J.dst + (size_t)mat * J.dst_stride + (size_t)(f - (long long)mat * per) * 16) = make_uint4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ void pack_tile16_item(const BwdPackJob &J, long long f)
{
    const int NT = J.N / 32;
    const long long per = (long long)(J.K / 16) * NT * 64;
    const int mat = (int)(f / per);
    long long r = f - (long long)mat * per;
    const int lane = (int)(r % 64);
    r /= 64;
    const int nt = (int)(r % NT), kt = (int)(r / NT);
    const int row = 16 * kt + (lane & 15), col = 32 * nt + 8 * (lane >> 4);   // column stride 1
    const bf16_t *src = J.src + (size_t)mat * J.src_stride + (size_t)row * J.rs + col;
    uint4 o = make_uint4(0, 0, 0, 0);
    if (row < J.Kv) {
        if (((uintptr_t)src & 15) == 0) o = *(const uint4 *)src;
        else o = make_uint4(src[0] | ((uint32_t)src[1] << 16), src[2] | ((uint32_t)src[3] << 16), src[4] | ((uint32_t)src[5] << 16),
                            src[6] | ((uint32_t)src[7] << 16));
    }
    *(uint4 *)(J.dst + (size_t)mat * J.dst_stride + (size_t)(f - (long long)mat * per) * 16) = o;
}

__device__ __forceinline__ void pack_bias_item(const BwdPackJob &J, long long t)
{
    // K = values per matrix, N = padded count
    const int mat = (int)(t / J.N), i = (int)(t - (long long)mat * J.N);
    ((float *)(J.dst + (size_t)mat * J.dst_stride))[i] = i < J.K ? bf16_to_f32(J.src[(size_t)mat * J.src_stride + i]) : 0.f;
}

constexpr int kPackThreads = 256;
__device__ __forceinline__ void capacity_sums(const CapSums &C)
{
    __shared__ unsigned long long sums[64];
    if (threadIdx.x < 64) sums[threadIdx.x] = 0ull;
    __syncthreads();
    auto add = [&](int expert, float prob) {
        const int e = min(max(expert, 0), C.E - 1);
        const float p = fminf(fmaxf(prob, 0.f), 1.f);
        atomicAdd(&sums[e], (unsigned long long)__float2ll_rn(p * C.scale));
    };
    // Four assignments a load, sixteen in flight: a block is a chain of loads, and there are at most kCapBlocks of them.  (idx and pk are regions
    // of the forward's workspace, 256-byte aligned.)
    const long long quads = C.Na / 4, first = (long long)blockIdx.x * kPackThreads + threadIdx.x;
#pragma unroll 4
    for (long long q = first; q < quads; q += (long long)C.blocks * kPackThreads) {
        const int4 e = ((const int4 *)C.idx)[q];
        const float4 p = ((const float4 *)C.pk)[q];
        add(e.x, p.x);
        add(e.y, p.y);
        add(e.z, p.z);
        add(e.w, p.w);
    }
    if (first < C.Na - quads * 4) add(C.idx[quads * 4 + first], C.pk[quads * 4 + first]);
    __syncthreads();
    if (threadIdx.x < C.E) C.slots[(size_t)blockIdx.x * C.E + threadIdx.x] = sums[threadIdx.x];
}

__global__ __launch_bounds__(kPackThreads) void bwd_pack_jobs_kernel(BwdPackJobs jobs, CapSums cap)
{
    if ((int)blockIdx.x < cap.blocks) {
        capacity_sums(cap);
        return;
    }
    long long f = (long long)(blockIdx.x - cap.blocks) * kPackThreads + threadIdx.x;
    for (int q = 0; q < jobs.count; ++q) {   // the jobs' items are numbered one job after the other
        const BwdPackJob &J = jobs.job[q];
        if (f < J.items) {
            if (J.kind == kPackLayer1) pack_layer1_item(J, f);
            else if (J.kind == kPackBias) pack_bias_item(J, f);
            else if (J.kind == kPackTile16) pack_tile16_item(J, f);
            else pack_chain_item(J, f);
            return;
        }
        f -= J.items;
    }
}

BwdPackJob bwd_pack_job(int kind, const void *src, int K, int Kv, int N, int Nv, size_t rs, size_t cs, size_t src_stride,
                        char *dst, size_t dst_stride, int nmat)
{
    BwdPackJob J;
    J.kind = kind;
    J.src = (const bf16_t *)src;
    J.K = K; J.Kv = Kv; J.N = N; J.Nv = Nv;
    J.rs = rs; J.cs = cs; J.src_stride = src_stride;
    J.dst = dst; J.dst_stride = dst_stride;
    if (kind == kPackLayer1) J.items = (long long)nmat * (N / 32) * (K / 16) * 64;
    else if (kind == kPackBias) J.items = (long long)nmat * N;
    else if (kind == kPackTile16) J.items = (long long)nmat * (K / 16) * (N / 32) * 64;
    else J.items = (long long)nmat * (K / 32) * 2 * (N / 32) * 64;
    return J;
}

hipError_t bwd_pack_launch(const BwdPackJobs &jobs, const CapSums &cap, hipStream_t s)
{
    long long total = 0;
    for (int q = 0; q < jobs.count; ++q) total += jobs.job[q].items;
    const long long blocks = (total + kPackThreads - 1) / kPackThreads + cap.blocks;
    if (blocks == 0) return hipSuccess;
    bwd_pack_jobs_kernel<<<(unsigned)blocks, kPackThreads, 0, s>>>(jobs, cap);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------- rows kernel, streamed
// For the experts that the fused kernel does not take: a block takes tiles of WAVES x 32 rows of ONE expert and streams the
// fragments through LDS in chunks of hc hidden tiles per row tile, the dL/dx accumulators staying in registers across the
// chunks.  Eight wavefronts (two per SIMD); four at width 192, whose rows and accumulators take more than half a SIMD's
// registers.
template <int DS> constexpr int kBmTileWaves = DS <= 128 ? 8 : 4;
template <int DS>
__global__ __launch_bounds__(kBmTileWaves<DS> * 64) void bwd_rows_streamed_mfma_kernel(
    const bf16_t *__restrict__ x, const bf16_t *__restrict__ dout, const float *__restrict__ pk,
    const int32_t *__restrict__ offsets, const int32_t *__restrict__ perm, const char *__restrict__ packed,
    size_t e_stride, size_t off_w2r, size_t off_w1c, size_t off_b1, int He, int hc, int E, int k,
    float *__restrict__ dxrow, float *__restrict__ dpk)
{
    constexpr int KS = SliceTiles<DS>::KS, OT = SliceTiles<DS>::OT, THREADS = kBmTileWaves<DS> * 64, kBmTileRows = kBmTileWaves<DS> * 32;
    static_assert(DS % 32 == 0, "whole tiles of features");
    const int HT = He / 32, nchunks = HT / hc;   // hc divides HT
    extern __shared__ __align__(16) char lds[];
    uint4 *w1f = (uint4 *)lds;                          // [hc][KS][64]
    uint4 *w2r = w1f + (size_t)hc * KS * 64;            // [hc][KS][64]
    uint4 *w1c = w2r + (size_t)hc * KS * 64;            // [hc][2][OT][64]
    float *b1s = (float *)(w1c + (size_t)hc * 2 * OT * 64);   // [He]
    int *tile_prefix = (int *)(b1s + He);               // [E + 1]

    const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid == 0) {
        int run = 0;
        for (int e = 0; e < E; ++e) {
            tile_prefix[e] = run;
            run += (offsets[e + 1] - offsets[e] + kBmTileRows - 1) / kBmTileRows;
        }
        tile_prefix[E] = run;
    }
    __syncthreads();
    const int total = tile_prefix[E];
    const int per_block = (total + (int)gridDim.x - 1) / (int)gridDim.x;
    const int t_begin = (int)blockIdx.x * per_block;
    const int t_end = min(total, t_begin + per_block);

    int cur_e = -1, e = 0;
    for (int t = t_begin; t < t_end; ++t) {
        while (tile_prefix[e + 1] <= t) ++e;
        const int row_begin = offsets[e] + (t - tile_prefix[e]) * kBmTileRows;
        const int row_end = offsets[e + 1];
        const char *ew = packed + (size_t)e * e_stride;
        const int row = row_begin + wave * 32 + j;
        const bool valid = row < row_end;
        const int a = perm[valid ? row : row_begin];
        const long long n = a / k;
        const float p = valid ? pk[a] : 0.f, half_p = 0.5f * p;
        const uint4 *xr = (const uint4 *)(x + n * DS), *gr = (const uint4 *)(dout + n * DS);
        bf16x8 xb[KS], gb[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            xb[ks] = load_row_piece<DS>(xr, ks, g);
            gb[ks] = load_row_piece<DS>(gr, ks, g);
        }
        f32x16 dx[OT];
#pragma unroll
        for (int ot = 0; ot < OT; ++ot)
#pragma unroll
            for (int i = 0; i < 16; ++i) dx[ot][i] = 0.f;
        float dps[8];   // dL/dp: eight sums side by side, a single chain over the hidden units would round more than a tree
#pragma unroll
        for (int i = 0; i < 8; ++i) dps[i] = 0.f;
        for (int ch = 0; ch < nchunks; ++ch) {
            __syncthreads();   // everyone is done with the previous contents
            // (eight pieces in flight per thread: one at a time took 1.08 ms at width 128, 1 048 576 rows, He 512, now 0.97)
            stage_to_lds<THREADS, 8>(ew + (size_t)ch * hc * KS * 1024, w1f, hc * KS * 64, tid);
            stage_to_lds<THREADS, 8>(ew + off_w2r + (size_t)ch * hc * KS * 1024, w2r, hc * KS * 64, tid);
            stage_to_lds<THREADS, 8>(ew + off_w1c + (size_t)ch * hc * 2 * OT * 1024, w1c, hc * 2 * OT * 64, tid);
            if (e != cur_e && ch == 0) {
                const float *gb1 = (const float *)(ew + off_b1);
                for (int i = tid; i < He; i += THREADS) b1s[i] = gb1[i];
            }
            __syncthreads();
#pragma unroll 1
            for (int hl = 0; hl < hc; ++hl) {
                const int ht = ch * hc + hl;
                f32x16 u, da;
#pragma unroll
                for (int i = 0; i < 16; ++i) u[i] = da[i] = 0.f;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    u = mfma_bf16(__builtin_bit_cast(bf16x8, w1f[(hl * KS + ks) * 64 + lane]), xb[ks], u);
                    da = mfma_bf16(__builtin_bit_cast(bf16x8, w2r[(hl * KS + ks) * 64 + lane]), gb[ks], da);
                }
                constexpr int TERMS = backward_terms(DS);   // of p dz
                uint32_t pd[2][TERMS][4];   // p dz by K-step of the second product; terms, the largest first
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) {
                    const f32x4 bb = *(const f32x4 *)(b1s + ht * 32 + 8 * qq + 4 * g);
                    float z[4], act[4], slope[4], pdz[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) z[c] = fmaf(p, u[4 * qq + c], bb[c]);
                    twice_gelu4(z, act, slope);
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float dz = da[4 * qq + c] * slope[c];   // twice dL/dz
                        dps[4 * (qq & 1) + c] = fmaf(dz, u[4 * qq + c], dps[4 * (qq & 1) + c]);
                        pdz[c] = half_p * dz;
                    }
                    split_terms<TERMS>(pdz, pd[qq >> 1], 2 * (qq & 1));
                }
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int ot = 0; ot < OT; ++ot) {
                        const bf16x8 wf = __builtin_bit_cast(bf16x8, w1c[((hl * 2 + s) * OT + ot) * 64 + lane]);
#pragma unroll
                        for (int t = TERMS - 1; t >= 0; --t)   // small terms first
                            dx[ot] = mfma_bf16(wf, __builtin_bit_cast(bf16x8, make_uint4(pd[s][t][0], pd[s][t][1], pd[s][t][2], pd[s][t][3])), dx[ot]);
                    }
            }
        }
        cur_e = e;
        float dp = ((dps[0] + dps[1]) + (dps[2] + dps[3])) + ((dps[4] + dps[5]) + (dps[6] + dps[7]));
        dp += __shfl_xor(dp, 32);
        if (valid) {
            if (g == 0) dpk[a] = 0.5f * dp;
            float *dst = dxrow + (size_t)row * DS;
#pragma unroll
            for (int ot = 0; ot < OT; ++ot)
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) {
                    const f32x4 v = {dx[ot][4 * qq], dx[ot][4 * qq + 1], dx[ot][4 * qq + 2], dx[ot][4 * qq + 3]};
                    *(f32x4 *)(dst + ot * 32 + 8 * qq + 4 * g) = v;
                }
        }
    }
}

// ------------------------------------------------------------------------------------------------------ host
// Hidden tiles per chunk of the streamed rows kernel: the largest divisor of HT whose fragments fit, and its LDS bytes.
static int streamed_chunk(int KS, int OT, int He, int E, size_t *lds)
{
    const int HT = He / 32;
    const size_t per_ht = (size_t)(2 * KS + 2 * OT) * 1024, fixed = (size_t)He * 4 + (size_t)(E + 1) * 4 + 64;
    const size_t want = 140 * 1024, dev = (size_t)max_lds_per_block();
    const size_t budget = dev < want ? dev : want;
    int hc = 1;
    for (int c = HT; c >= 1; --c)
        if (HT % c == 0 && per_ht * c + fixed <= budget) {
            hc = c;
            break;
        }
    *lds = per_ht * hc + fixed;
    return hc;
}

bool backward_mfma_shape(const slicemoe_config &c)
{
    const int ds = c.d / c.S;
    const bool width = ds == 24 || ds == 48 || ds == 64 || ds == 96 || ds == 128 || ds == 192;
    if (c.dtype != SLICEMOE_BF16 || !width || c.He % 32 != 0 || (c.flags & SLICEMOE_FLAG_FORCE_GENERIC)) return false;
    // the rows kernel keeps an expert's biases in the LDS, beside at least one hidden tile's fragments: hidden widths up to about
    // 31 000 (slice width 192) to 37 000 (64); the fp32 kernels take any.  At 24 and 48, whose kernel keeps none, the limit (39 000) stays: nothing
    // wider has been measured there.
    size_t lds = 0;
    streamed_chunk((ds + 15) / 16, (ds + 31) / 32, c.He, c.E, &lds);
    return lds <= (size_t)max_lds_per_block();
}

size_t backward_mfma_packed_bytes(const slicemoe_config &c)
{
    return bwd_packed_layout(c).stride * (size_t)c.E;
}

template <int DS>
static hipError_t run_rows_mfma(const slicemoe_config &c, const BwdPacked &L, const void *h, const void *d_out, const float *pk,
                                const int32_t *offsets, const int32_t *perm, const char *packed, float *dxrow, float *dpk, hipStream_t s)
{
    const long long Na = (long long)c.T * c.S * c.k;
    constexpr int kTileRows = kBmTileWaves<DS> * 32;
    size_t lds = 0;
    const int hc = streamed_chunk(SliceTiles<DS>::KS, SliceTiles<DS>::OT, c.He, c.E, &lds);
    long long blocks = (Na + kTileRows - 1) / kTileRows + c.E;
    if (blocks > num_compute_units()) blocks = num_compute_units();
    auto rows = bwd_rows_streamed_mfma_kernel<DS>;
    const hipError_t e = grant_dynamic_lds((const void *)rows, lds);
    if (e != hipSuccess) return e;
    rows<<<(int)blocks, kBmTileWaves<DS> * 64, lds, s>>>((const bf16_t *)h, (const bf16_t *)d_out, pk, offsets, perm, packed, L.stride,
                                                         L.w2r, L.w1c, L.b1, c.He, hc, c.E, c.k, dxrow, dpk);
    return hipGetLastError();
}

void backward_expert_pack_jobs(const slicemoe_config &c, const BackwardWeightsPlan &W, const slicemoe_weights &w, void *packed, BwdPackJobs &jobs)
{
    const int He = c.He, E = c.E, ds = c.d / c.S, dsK = (ds + 15) / 16 * 16, dsN = (ds + 31) / 32 * 32;
    const BwdPacked L = bwd_packed_layout(c);
    char *pb = (char *)packed;
    const size_t wstride = (size_t)ds * He;
    BwdPackJob *J = jobs.job + jobs.count;
    jobs.count += W.onepass ? 3 : 4;
    // w1f: the [ds, He] matrix W1 itself; w2r: the [ds, He] matrix M[c][hidden] = W2[hidden][c]
    J[0] = bwd_pack_job(kPackLayer1, w.W1, dsK, ds, He, He, (size_t)He, 1, wstride, pb + L.w1f, L.stride, E);
    J[1] = bwd_pack_job(kPackLayer1, w.W2, dsK, ds, He, He, 1, (size_t)ds, wstride, pb + L.w2r, L.stride, E);
    J[2] = bwd_pack_job(kPackBias, w.b1, He, He, He, He, 0, 0, (size_t)He, pb + L.b1, L.stride, E);
    if (W.onepass) return;
    // w1d: W1 in 16-feature tiles.  w1c: the [He, ds] matrix M[hidden][c] = W1[c][hidden], contraction over the hidden units
    // in accumulator order
    if (W.fused)
        J[3] = bwd_pack_job(kPackTile16, w.W1, dsK, ds, He, He, (size_t)He, 1, wstride, pb + L.w1d, L.stride, E);
    else J[3] = bwd_pack_job(kPackChain, w.W1, He, He, dsN, ds, 1, (size_t)He, wstride, pb + L.w1c, L.stride, E);
}

// Runs the kernels on the backward copies of the expert weights in `packed` (backward_expert_pack_jobs, launched on s before).
// part holds W.slots slots of slot_floats floats, W = backward_weights_plan(c).  When the weight gradients come from a kernel of
// their own it runs on the side stream (if there is one), from the moment the repacked weights are there.
hipError_t launch_backward_expert_mfma(const slicemoe_config &c, const BackwardWeightsPlan &W, const void *h, const void *d_out,
                                       const float *pk, const int32_t *offsets, const int32_t *perm, void *packed,
                                       size_t slot_floats, float *dxrow, float *dpk, float *part, hipStream_t s,
                                       const SideStream *side)
{
    const int ds = c.d / c.S;
    const BwdPacked L = bwd_packed_layout(c);
    const char *pb = (const char *)packed;
    hipError_t e;
    if (W.onepass) return launch_backward_expert_onepass(c, W, L, h, d_out, pk, offsets, perm, pb, slot_floats, part, dxrow, dpk, s);
    if (!W.fused) {
        if (side != nullptr) {
            if ((e = hipEventRecord(side->fork, s)) != hipSuccess) return e;
            if ((e = hipStreamWaitEvent(side->stream, side->fork, 0)) != hipSuccess) return e;
        }
        e = ds == 64 ? run_rows_mfma<64>(c, L, h, d_out, pk, offsets, perm, pb, dxrow, dpk, s)
          : ds == 96 ? run_rows_mfma<96>(c, L, h, d_out, pk, offsets, perm, pb, dxrow, dpk, s)
          : ds == 128 ? run_rows_mfma<128>(c, L, h, d_out, pk, offsets, perm, pb, dxrow, dpk, s)
                      : run_rows_mfma<192>(c, L, h, d_out, pk, offsets, perm, pb, dxrow, dpk, s);
        if (e != hipSuccess) return e;
    }
    return launch_backward_weights(c, W, L, h, d_out, pk, offsets, perm, pb, slot_floats, part, dxrow, dpk,
                                   !W.fused && side != nullptr ? side->stream : s);
}

}  // namespace slicemoe
