// Backward pass on fp32 arithmetic, for every shape the bf16 matrix-core kernels do not take (fp32 storage, other slice
// widths, forced generic): gradients by the chain rule as described in backward.hip, any shape within the library limits,
// either storage type.  The contractions run on the fp32 matrix instruction (32 x 32 x 2: operands, products and sums
// fp32), in the layout of backward_weights_mfma.hip: a block of eight wavefronts works on 32 rows (slices), a wavefront owns
// one 32-wide hidden tile, lane = hidden unit, registers = rows.  What is formed there is directly the operand of the weight
// gradients (contraction over rows); for the gradients of the rows (contraction over the hidden units) it goes through the
// LDS.  Slice features are taken in chunks of 32 OTC columns, one block per chunk (grid.y), each chunk recomputing the
// shared quantities; hidden widths above 256 in groups that a block works through in turn, the same thread adding each
// group's part of dL/dx and dL/dp to what it wrote before.  Nothing is added in an order that changes from run to run.
//
// Bound: the matrix instruction (64 cycles; 160 per hidden tile and unit at ds = 64, 8.5 us for the two wavefronts of a SIMD) and,
// for the small batches these shapes run at, latency.  Where a block has the whole width and whole quads (AHEAD: 32 or 64 columns,
// He a multiple of 32), the weights are requested ahead without conditions: the first batch with the rows, the next one and dL/dx's
// while matrix instructions run.  Elsewhere, with a test per load, a batch at its use.  8000 rows, ds = 64, He = 256, 8 experts: 33 ->
// 27 us; 32 768 rows (a step's backward): 188 -> 156; ragged widths, ds = 40, He = 100, 8000 rows: 123 -> 83 (bases of the LDS
// accesses in registers instead of an address per access, spilled, and the rows gathered without a barrier between their index and their load);
// router, 4000 slices, E = 8: 3.69 ms -> 26 us (one thread per hidden unit over 512 rows per block before).
#include "bwd_mfma.h"

namespace slicemoe {

constexpr int kGbThreads = 512, kGbWaves = 8, kGbRows = 32, kGbHidden = 256;
constexpr int kGbT = 33;   // row stride of 32-wide tiles: neighbouring rows in different banks

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// Four consecutive values p[0..3], those at or past `n` zero; vec: the address is aligned for one load.
template <typename T> struct Quad;
template <> struct Quad<float> {
    static __device__ __forceinline__ void load(const float *p, float (&v)[4])
    {
        const float4 q = *(const float4 *)p;
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    }
};
template <> struct Quad<bf16_t> {
    static __device__ __forceinline__ void load(const bf16_t *p, float (&v)[4])
    {
        const uint2 q = *(const uint2 *)p;
        v[0] = __uint_as_float(q.x << 16); v[1] = __uint_as_float(q.x & 0xffff0000u);
        v[2] = __uint_as_float(q.y << 16); v[3] = __uint_as_float(q.y & 0xffff0000u);
    }
};
__device__ __forceinline__ void store_quad(float *p, const float (&v)[4]) { *(float4 *)p = make_float4(v[0], v[1], v[2], v[3]); }
__device__ __forceinline__ void store_quad(bf16_t *p, const float (&v)[4])
{
#pragma unroll
    for (int c = 0; c < 4; ++c) Storage<bf16_t>::store(p + c, v[c]);
}
template <typename T> __device__ __forceinline__ void load_quad(const T *p, int n, bool vec, float (&v)[4])
{
    if (vec && n >= 4) {
        Quad<T>::load(p, v);
        return;
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = s < n ? Storage<T>::load(p + s) : 0.f;
}

// d/dz of the exact GELU z Phi(z): Phi(z) + z phi(z)
__device__ __forceinline__ float gelu_grad(float z, float *act)
{
    const float cdf = 0.5f * (1.f + erff(z * 0.70710678118654752f));
    *act = z * cdf;
    return cdf + z * expf(-0.5f * z * z) * 0.39894228040143267794f;
}

// ------------------------------------------------------------------------------------------------ experts
template <int OTC> struct GenericExpertLds {
    static constexpr int CC = 32 * OTC, XST = CC + 1;
    static constexpr size_t xs = 0, gs = xs + (size_t)kGbRows * XST, pz = gs + (size_t)kGbRows * XST;   // floats
    static constexpr size_t red = pz + (size_t)kGbHidden * kGbT, dps = red + (size_t)kGbWaves * kGbRows * kGbT;
    static constexpr size_t ps = dps + kGbWaves * kGbRows, total = ps + kGbWaves * kGbRows;
};

template <typename T, int OTC, bool AHEAD>
__global__ __launch_bounds__(kGbThreads) void bwd_expert_generic_kernel(
    const T *__restrict__ x, const T *__restrict__ dout, const float *__restrict__ pk,
    const int32_t *__restrict__ offsets, const int32_t *__restrict__ perm, int ds, int He, int E, int k,
    const T *__restrict__ W1, const T *__restrict__ b1, const T *__restrict__ W2, bool vec_ds, bool vec_he,
    float *__restrict__ dxrow, float *__restrict__ dpk, size_t slot_floats, float *__restrict__ part)
{
    typedef GenericExpertLds<OTC> L;
    constexpr int CC = L::CC, XST = L::XST, PARTS = kGbWaves / OTC;
    extern __shared__ __align__(16) float smem[];
    float *xs = smem + L::xs, *gs = smem + L::gs, *pz = smem + L::pz, *red = smem + L::red, *dps = smem + L::dps, *ps = smem + L::ps;
    const int tid = threadIdx.x, lane = tid & 63, jj = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nch = AHEAD ? 1 : (int)gridDim.y, own = AHEAD ? 0 : (int)blockIdx.y, own_c0 = own * CC, own_n = AHEAD ? CC : min(CC, ds - own_c0);
    const int off_lo = offsets[min(lane, E)], off_hi = offsets[min(lane + 1, E)];
    const RowAxis A = row_axis(off_hi - off_lo, kGbRows, 0, (int)gridDim.x, lane);
    const int p0 = (int)blockIdx.x * A.share, p1 = p0 + A.share;
    constexpr int ROWS = kGbThreads / CC, STAGED = kGbRows / ROWS;   // staging: a thread has one column of every ROWS-th row
    const int st_c = tid % CC, st_r = tid / CC;
    // LDS bases of a lane: what is added to them in the loops is known to the compiler and takes no register
    const float *xs_b = xs + jj * XST + g, *gs_b = gs + jj * XST + 4 * g, *xs_r = xs + 4 * g * XST + jj, *gs_r = gs + 4 * g * XST + jj, *ps_r = ps + wave * kGbRows + 4 * g;
    float *pz_w = pz + (wave * 32 + jj) * kGbT + 4 * g, *red_w = red + (wave * kGbRows + 4 * g) * kGbT + jj;
    // Values kb + 8 q + 4 g .. of a row of n, zero past it: `row` elements from the uniform p, so that an address is one register.  The rows of a
    // tile count from p, which has the tile's own 64-bit offset: 31 rows are below 4 GB (He up to 34 million fp32 values).
    auto quads_of = [&](const T *p, unsigned row, int kb, int n, bool vec, float (&b)[16]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float v[4];
            const int f = kb + 8 * q + 4 * g;
            const T *at = (const T *)((const char *)(p + kb + 8 * q) + (row + 4u * (unsigned)g) * (unsigned)sizeof(T));
            if (AHEAD) Quad<T>::load(at, v);
            else load_quad(at, n - f, vec, v);
#pragma unroll
            for (int s = 0; s < 4; ++s) b[4 * q + s] = v[s];
        }
    };

    for (int e = 0; e < E; ++e) {
        const int first = __builtin_amdgcn_readlane(A.first, e), steps = __builtin_amdgcn_readlane(A.steps, e);
        if (first >= p1) break;
        const int s_lo = max(0, p0 - first), s_hi = min(steps, p1 - first);
        if (s_hi <= s_lo) continue;
        const int row0 = __builtin_amdgcn_readlane(off_lo, e) + s_lo * kGbRows;
        const int nrows = min(__builtin_amdgcn_readlane(off_hi, e) - row0, (s_hi - s_lo) * kGbRows);
        const T *w1 = W1 + (size_t)e * ds * He, *w2 = W2 + (size_t)e * He * ds;
        float *slot = part + (size_t)((int)blockIdx.x + e) * slot_floats;
        float *pW1 = slot, *pW2 = pW1 + (size_t)ds * He, *pb1 = pW2 + (size_t)He * ds, *pb2 = pb1 + He;

        for (int h0 = 0; h0 < He; h0 += kGbHidden) {
            const int hid = h0 + wave * 32 + jj, hidc = min(hid, He - 1);
            const bool hok = hid < He;
            const float bias = Storage<T>::load(b1 + (size_t)e * He + hidc);
            f32x16 aW1[OTC], aW2[OTC];
#pragma unroll
            for (int ot = 0; ot < OTC; ++ot)
#pragma unroll
                for (int i = 0; i < 16; ++i) aW1[ot][i] = aW2[ot][i] = 0.f;
            float ab1 = 0.f, ab2 = 0.f;
            // operands of 32 of a chunk's features: column hid of W1, row hid of W2 (K-step s of quad q: features kb + 8 q + 4 g + s)
            auto first_layer = [&](int c0, int nf, int kb, float (&bu)[16], float (&bd)[16]) {
                const int tile = min(h0 + wave * 32, He - 1);   // (uniform)
                unsigned col = (unsigned)(g * He + hidc), row = (unsigned)(min(jj, He - 1 - tile) * ds);
                asm volatile("" : "+v"(col), "+v"(row));   // opaque: addresses are not kept in registers from one unit to the next
#pragma unroll
                for (int s = 0; s < 16; ++s) {
                    const T *at = (const T *)((const char *)(w1 + (size_t)(c0 + kb + 2 * s) * He) + col * (unsigned)sizeof(T));
                    if (AHEAD) bu[s] = Storage<T>::load(at);
                    else bu[s] = kb + 2 * s + g < nf ? Storage<T>::load(at) : 0.f;
                }
                quads_of(w2 + (size_t)tile * ds + c0, row, kb, nf, vec_ds, bd);
            };
            int assigned = perm[row0 + min(jj, nrows - 1)];   // of row jj of the unit, in every wavefront
            for (int r0 = 0; r0 < nrows; r0 += kGbRows) {
                const int rows = min(kGbRows, nrows - r0), mine = assigned;
                f32x16 u, da;
#pragma unroll
                for (int i = 0; i < 16; ++i) u[i] = da[i] = 0.f;
                for (int i = 1; i <= nch; ++i) {   // the block's own columns last: they stay for the weight gradients
                    const int c0 = AHEAD ? 0 : (own + i) % nch * CC, nf = AHEAD ? CC : min(CC, ds - c0);
                    float bu[AHEAD ? 2 : 1][16], bd[AHEAD ? 2 : 1][16];
                    if (AHEAD) first_layer(c0, nf, 0, bu[0], bd[0]);
                    float xv[STAGED], gv[STAGED], pv = 0.f;
                    {
                        const int n = mine / k;
                        if (i == 1) pv = pk[mine];
#pragma unroll
                        for (int q = 0; q < STAGED; ++q) {
                            const size_t at = (size_t)__shfl(n, st_r + q * ROWS) * ds + c0 + min(st_c, nf - 1);
                            xv[q] = Storage<T>::load(x + at);
                            gv[q] = Storage<T>::load(dout + at);
                        }
                    }
                    if (i == 1) assigned = perm[row0 + min(r0 + kGbRows + jj, nrows - 1)];
                    __syncthreads();   // everyone is done with what was there
#pragma unroll
                    for (int q = 0; q < STAGED; ++q) {
                        const int r = st_r + q * ROWS;
                        xs[r * XST + st_c] = st_c < nf ? xv[q] : 0.f;
                        gs[r * XST + st_c] = st_c < nf && r < rows ? gv[q] : 0.f;   // rows past the end add nothing
                    }
                    if (i == 1) ps[wave * kGbRows + jj] = jj < rows ? pv : 0.f;   // a wavefront's own copy
                    __syncthreads();
                    // 32 features at a time: sixteen weights of each product in flight, then sixteen matrix instructions of each
#pragma unroll
                    for (int t = 0; t < OTC; ++t) {
                        const int kb = 32 * t, at = AHEAD ? t & 1 : 0;
                        if (kb >= nf) break;
                        if (!AHEAD) first_layer(c0, nf, kb, bu[0], bd[0]);
                        else if (t + 1 < OTC) first_layer(c0, nf, kb + 32, bu[(t + 1) & 1], bd[(t + 1) & 1]);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int s = 0; s < 16; ++s) {
                            u = mfma_f32(xs_b[kb + 2 * s], bu[at][s], u);
                            da = mfma_f32(gs_b[kb + 8 * (s >> 2) + (s & 3)], bd[at][s], da);
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                float bx[AHEAD ? OTC : 1][16];   // of dL/dx, requested ahead of the activations
                const int dx_t = wave % OTC, dx_k0 = wave / OTC * (kGbHidden / PARTS), dx_k1 = min(dx_k0 + kGbHidden / PARTS, He - h0);
                const int dx_tile = min(32 * dx_t, own_n - 1);
                const T *wf = w1 + (size_t)(own_c0 + dx_tile) * He + h0;
                unsigned dx_row = (unsigned)min(jj, own_n - 1 - dx_tile) * (unsigned)He;
                asm volatile("" : "+v"(dx_row));
                if (AHEAD) {
#pragma unroll
                    for (int q = 0; q < OTC; ++q) quads_of(wf, dx_row, min(dx_k0 + 32 * q, He - h0 - 32), He - h0, vec_he, bx[q]);   // (those past the end are not used)
                }
                __builtin_amdgcn_sched_barrier(0);
                float du[8];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int row = acc_feature(i, 0);   // and 4 g more, in the bases
                    const float p = ps_r[row], z = fmaf(p, u[i], bias);
                    float act;
                    const float gg = gelu_grad(z, &act), dz = hok ? da[i] * gg : 0.f, pdz = p * dz;
                    du[i & 7] = i < 8 ? dz * u[i] : sum_over_row_pair(du[i & 7], dz * u[i]);
                    ab1 += dz;
                    pz_w[row] = pdz;
#pragma unroll
                    for (int ot = 0; ot < OTC; ++ot) {
                        aW1[ot] = mfma_f32(xs_r[row * XST + 32 * ot], pdz, aW1[ot]);   // [feature][hidden unit]: lane = hidden unit
                        aW2[ot] = mfma_f32(act, gs_r[row * XST + 32 * ot], aW2[ot]);   // [hidden unit][feature]: lane = feature
                    }
                    if (i & 1) __builtin_amdgcn_sched_barrier(0);   // two elements at a time: more would not fit the registers
                }
                sum_over_hidden(du);
                if ((lane & 3) == 0) *(float2 *)(dps + wave * kGbRows + hidden_sum_row(lane)) = make_float2(du[0], du[1]);
                if (h0 == 0 && tid < own_n)
                    for (int r = 0; r < rows; ++r) ab2 += gs[r * XST + tid];
                __syncthreads();
                {   // dL/dx, own columns: lane = feature, registers = rows; the hidden units of a tile over PARTS wavefronts
                    f32x16 dx;
#pragma unroll
                    for (int i = 0; i < 16; ++i) dx[i] = 0.f;
#pragma unroll
                    for (int q = 0; q < OTC; ++q) {
                        const int kb = dx_k0 + 32 * q;
                        if (kb >= dx_k1) break;
                        __builtin_amdgcn_sched_barrier(0);
                        const float *pz_b = pz + (kb + 4 * g) * kGbT + jj;
                        if (!AHEAD) quads_of(wf, dx_row, kb, He - h0, vec_he, bx[0]);
#pragma unroll
                        for (int s = 0; s < 16; ++s) dx = mfma_f32(pz_b[(8 * (s >> 2) + (s & 3)) * kGbT], bx[AHEAD ? q : 0][s], dx);
                    }
#pragma unroll
                    for (int i = 0; i < 16; ++i) red_w[acc_feature(i, 0) * kGbT] = dx[i];
                }
                __syncthreads();
                for (int t = tid; t < rows * own_n; t += kGbThreads) {
                    const int r = t / own_n, f = t - r * own_n;
                    float v = 0.f;
#pragma unroll
                    for (int q = 0; q < PARTS; ++q) v += red[((q * OTC + (f >> 5)) * kGbRows + r) * kGbT + (f & 31)];
                    float *dst = dxrow + (size_t)(row0 + r0 + r) * ds + own_c0 + f;   // the same thread wrote it for the group before
                    *dst = h0 > 0 ? *dst + v : v;
                }
                if (own == 0 && tid < rows) {
                    float v = 0.f;
#pragma unroll
                    for (int w = 0; w < kGbWaves; ++w) v += dps[w * kGbRows + tid];
                    dpk[mine] = h0 > 0 ? dpk[mine] + v : v;
                }
            }
            // ---- this segment's slot: dW1 [ds][He] | dW2 [He][ds] | db1 [He] | db2 [ds]; every element is written once
            int jo = jj, go = g;   // opaque copies: the addresses are made here, not kept in registers through the loop above
            asm volatile("" : "+v"(jo), "+v"(go));
#pragma unroll
            for (int ot = 0; ot < OTC; ++ot)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int f = 32 * ot + acc_feature(i, go), ho = h0 + wave * 32 + jo, hr = h0 + wave * 32 + acc_feature(i, go);
                    if (hok && f < own_n) pW1[(size_t)(own_c0 + f) * He + ho] = aW1[ot][i];
                    if (hr < He && 32 * ot + jo < own_n) pW2[(size_t)hr * ds + own_c0 + 32 * ot + jo] = aW2[ot][i];
                }
            ab1 += __shfl_xor(ab1, 32);
            if (own == 0 && g == 0 && hok) pb1[hid] = ab1;
            if (h0 == 0 && tid < own_n) pb2[own_c0 + tid] = ab2;
        }
    }
}

// ------------------------------------------------------------------------------------------------ router
// Hr <= 256 and E <= 64.  The hidden layer is recomputed by plain multiply-add chains in a fixed order over the features (its
// sign decides what the ReLU lets through): four hidden units and four slices per thread, weights and slices from LDS.
// AHEAD (256 hidden units, whole chunks of columns, whole octets of experts, everything aligned for quads): each phase's
// operands are requested, without conditions, before the phase in front of it -- the softmax's and the logits' with the slices, the
// expert path's rows and dL/dh's weights before the weight gradients -- and dL/dh leaves as one quad per thread.  A unit of 32
// slices is a chain of eight phases with a barrier between them, and half of its time was the latency of their loads: 4000
// slices, ds = 64, E = 8: 39 -> 26 us; 16 384 slices (a step's backward): 156 -> 137.  (It takes all 256 registers and spills 12, of which nine are
// reloaded in every unit; the instance without AHEAD spills none and is the slower one all the same.)
constexpr int kGrFeat = 64;   // features at a time, and columns of a block
struct GenericRouterLds {   // floats
    static constexpr size_t xT = 0, w = xT + (size_t)kGrFeat * 36, us = w + (size_t)kGrFeat * kGbHidden;   // us: [32][257] u, then [256][33] dL/du
    static constexpr size_t dgs = us + (size_t)kGbHidden * kGbT, red = dgs + (size_t)kGbRows * 65;
    static constexpr size_t total = red + (size_t)kGbWaves * kGbRows * kGbT;
};

template <typename T, bool AHEAD>
__global__ __launch_bounds__(kGbThreads) void bwd_router_generic_kernel(
    const T *__restrict__ x, long long Ns, int ds, int Hr, int E, int k,
    const T *__restrict__ Wr1, const T *__restrict__ br1, const T *__restrict__ Wr2, const T *__restrict__ br2,
    const float *__restrict__ noise, float sigma, float inv_tau, const float *__restrict__ drop_u, float rate,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ inv, const float *__restrict__ dpk,
    CapLoss cap, const float *__restrict__ dxrow, T *__restrict__ dh, int units_per_block, bool vec_hr, bool vec_e,
    float *__restrict__ part, size_t slot_floats)
{
    typedef GenericRouterLds L;
    constexpr int OTC = kGrFeat / 32, PARTS = kGbWaves / OTC, UST = kGbHidden + 1, GST = 65;
    extern __shared__ __align__(16) float smem[];
    float *xT = smem + L::xT, *ws = smem + L::w, *us = smem + L::us, *dgs = smem + L::dgs, *red = smem + L::red;
    const int tid = threadIdx.x, lane = tid & 63, jj = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nch = (int)gridDim.y, own = (int)blockIdx.y, own_c0 = own * kGrFeat, own_n = min(kGrFeat, ds - own_c0);
    const long long n_begin = (long long)blockIdx.x * units_per_block * kGbRows;
    const long long n_end = min(Ns, n_begin + (long long)units_per_block * kGbRows);
    __shared__ float capg_s[64];
    if (cap.slots != nullptr) {
        capacity_part<kGbWaves>(cap, E, tid, (unsigned long long *)us);
        __syncthreads();
        capacity_derivatives<kGbWaves>(cap, E, tid, (const unsigned long long *)us, capg_s);
        __syncthreads();
    }
    const int ET = (E + 31) / 32, hid = wave * 32 + jj, hidc = min(hid, Hr - 1);
    const bool hok = hid < Hr, quads = (ds & 3) == 0;

    f32x16 aW1[OTC], aW2[2];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        aW1[0][i] = aW1[1][i] = 0.f;
        aW2[0][i] = aW2[1][i] = 0.f;
    }
    float ab1 = 0.f, ab2 = 0.f;
    constexpr int STAGED = kGbRows * kGrFeat / kGbThreads, ROWS = kGbThreads / kGrFeat;   // a thread has one column of every ROWS-th slice
    const int st_c = tid % kGrFeat, st_r = tid / kGrFeat;
    // LDS bases of a lane (see the expert kernel)
    const float *u_r = us + 4 * g * UST + hid, *dg_b = dgs + jj * GST + 4 * g, *dg_r = dgs + 4 * g * GST + jj, *xT_r = xT + jj * 36 + 4 * g;
    float *du_w = us + hid * kGbT + 4 * g, *red_w = red + (wave * kGbRows + 4 * g) * kGbT + jj;
    auto request_x = [&](long long n0, int rows, int c0, int nf, float (&v)[STAGED]) {
#pragma unroll
        for (int q = 0; q < STAGED; ++q) v[q] = Storage<T>::load(x + (n0 + min(st_r + q * ROWS, rows - 1)) * ds + c0 + min(st_c, nf - 1));
    };
    auto stage_x = [&](int rows, int nf, const float (&v)[STAGED]) {
#pragma unroll
        for (int q = 0; q < STAGED; ++q) {
            const int r = st_r + q * ROWS;
            xT[st_c * 36 + r] = r < rows && st_c < nf ? v[q] : 0.f;
        }
    };

    for (long long n0 = n_begin; n0 < n_end; n0 += kGbRows) {
        const int rows = (int)min((long long)kGbRows, n_end - n0);
        unsigned here = 0;   // opaque: what is the same for every unit is requested in each, not kept in registers through all of them
        asm volatile("" : "+v"(here));
        // the slice and the experts of this thread in the softmax: everything that it reads there is requested here
        const int sm_r = tid >> 4, sm_l = tid & 15;
        const long long sm_n = n0 + min(sm_r, rows - 1);
        const long long sm_a = sm_n * k + min(sm_l, k - 1);   // lane l has assignment l
        const int sm_idx = idx[sm_a], sm_inv = inv[sm_a];
        const float sm_d = dpk[sm_a], sm_u = rate > 0.f ? drop_u[sm_a] : 0.f;
        float sm_noise[4], sm_b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) sm_b[i] = Storage<T>::load(br2 + (min(sm_l + 16 * i, E - 1) + here));
        if (noise != nullptr)
#pragma unroll
            for (int i = 0; i < 4; ++i) sm_noise[i] = noise[sm_n * E + min(sm_l + 16 * i, E - 1)];
        // ---- hidden layer: hidden units 4 lane .., slices 4 wave ..
        float lw[16];      // of the logits: 32 hidden units of Wr2's column e
        auto second_layer = [&](int kb, float (&b)[16]) {
            const int e = min(32 * (wave % ET) + jj, E - 1);
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                const T *at = (const T *)((const char *)(Wr2 + (size_t)(kb + 2 * s) * E) + ((unsigned)(g * E + e) + here) * (unsigned)sizeof(T));
                if (AHEAD) b[s] = Storage<T>::load(at);
                else b[s] = kb + 2 * s + g < Hr ? Storage<T>::load(at) : 0.f;
            }
        };
        float acc[4][4];   // [slice][hidden unit]
        float bias[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) bias[c] = AHEAD || 4 * lane + c < Hr ? Storage<T>::load(br1 + (4 * lane + here) + c) : 0.f;
        for (int ch = 0; ch < nch; ++ch) {
            const int c0 = ch * kGrFeat, nf = min(kGrFeat, ds - c0);
            if (AHEAD && ch == nch - 1) second_layer(wave / ET * (kGbHidden / (kGbWaves / ET)), lw);
            float xv[STAGED];
            request_x(n0, rows, c0, nf, xv);
            const bool weights = nch > 1 || n0 == n_begin;
            if (AHEAD && weights) {   // every wavefront whole rows: a quad per lane, eight rows in flight
                constexpr int QUADS = kGrFeat / kGbWaves;
                float wv[QUADS][4];
#pragma unroll
                for (int q = 0; q < QUADS; ++q) Quad<T>::load(Wr1 + (size_t)(c0 + min(wave + q * kGbWaves, nf - 1)) * Hr + 4 * lane, wv[q]);
                __syncthreads();   // everyone is done with the features before
#pragma unroll
                for (int q = 0; q < QUADS; ++q) *(float4 *)(ws + (wave + q * kGbWaves) * kGbHidden + 4 * lane) = make_float4(wv[q][0], wv[q][1], wv[q][2], wv[q][3]);
            } else {
                __syncthreads();
                if (weights)
                    for (int t = tid; t < nf * kGbHidden; t += kGbThreads) {
                        const int f = t / kGbHidden, j = t % kGbHidden;
                        ws[t] = j < Hr ? Storage<T>::load(Wr1 + (size_t)(c0 + f) * Hr + j) : 0.f;
                    }
            }
            stage_x(rows, nf, xv);
            __syncthreads();
            if (ch == 0)
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[r][c] = bias[c];
            if (quads) {
                for (int f = 0; f < nf; f += 4) {
                    float4 xq[4], wq[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        xq[q] = *(const float4 *)(xT + (f + q) * 36 + 4 * wave);
                        wq[q] = *(const float4 *)(ws + (f + q) * kGbHidden + 4 * lane);
                    }
#pragma unroll
                    for (int q = 3; q >= 0; --q) {   // (the last of four features first)
                        const float xr[4] = {xq[q].x, xq[q].y, xq[q].z, xq[q].w}, wc[4] = {wq[q].x, wq[q].y, wq[q].z, wq[q].w};
#pragma unroll
                        for (int r = 0; r < 4; ++r)
#pragma unroll
                            for (int c = 0; c < 4; ++c) acc[r][c] = fmaf(xr[r], wc[c], acc[r][c]);
                    }
                }
            } else {
                for (int f = 0; f < nf; ++f) {
                    const float4 xq = *(const float4 *)(xT + f * 36 + 4 * wave), wq = *(const float4 *)(ws + f * kGbHidden + 4 * lane);
                    const float xr[4] = {xq.x, xq.y, xq.z, xq.w}, wc[4] = {wq.x, wq.y, wq.z, wq.w};
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int c = 0; c < 4; ++c) acc[r][c] = fmaf(xr[r], wc[c], acc[r][c]);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) us[(4 * wave + r) * UST + 4 * lane + c] = fmaxf(acc[r][c], 0.f);
        __syncthreads();
        if (nch > 1) {   // the block's own columns, for dWr1
            float xv[STAGED];
            request_x(n0, rows, own_c0, own_n, xv);
            stage_x(rows, own_n, xv);
        }
        {   // ---- logits: lane = expert, registers = slices; the hidden units of a 32-expert tile over 8 / ET wavefronts
            const int per = kGbHidden / (kGbWaves / ET), k0 = wave / ET * per;
            f32x16 lg;
#pragma unroll
            for (int i = 0; i < 16; ++i) lg[i] = 0.f;
            for (int kb = k0; kb < k0 + per; kb += 32) {
                if (!AHEAD || kb != k0) second_layer(kb, lw);
                const float *u_b = us + jj * UST + kb + g;
#pragma unroll
                for (int s = 0; s < 16; ++s) lg = mfma_f32(u_b[2 * s], lw[s], lg);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) red_w[acc_feature(i, 0) * kGbT] = lg[i];
        }
        __syncthreads();
        float dw[AHEAD ? 4 : 1][4];   // of dL/du: the first 32 experts of Wr2's row hid
        if (AHEAD)
#pragma unroll
            for (int q = 0; q < 4; ++q) Quad<T>::load((const T *)((const char *)(Wr2 + min(8 * q, E - 8)) + ((unsigned)(hidc * E + 4 * g) + here) * (unsigned)sizeof(T)), dw[q]);
        {   // ---- softmax, back through the dropout's renormalisation, dL/dg: 16 lanes per slice, experts l, l + 16, ..
            const int r = sm_r, l = sm_l;
            float v[4], m = -INFINITY, den = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = l + 16 * i;
                v[i] = -INFINITY;
                if (e < E) {
                    float t = sm_b[i];
                    const float *at = red + ((e >> 5) * kGbRows + r) * kGbT + (e & 31);
#pragma unroll
                    for (int q = 0; q < 4; ++q) t += at[q * ET * kGbRows * kGbT];
                    if (ET == 1)
#pragma unroll
                        for (int q = 4; q < kGbWaves; ++q) t += at[q * kGbRows * kGbT];
                    if (noise != nullptr) t = fmaf(sigma, sm_noise[i], t);
                    v[i] = t;
                }
                m = fmaxf(m, v[i]);
            }
            for (int o = 8; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = l + 16 * i < E ? expf((v[i] - m) * inv_tau) : 0.f;
                den += v[i];
            }
            for (int o = 8; o > 0; o >>= 1) den += __shfl_xor(den, o);
            const float rden = 1.f / den;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] *= rden;   // softmax probability of every expert
            float psel[8], dpf[8];
            bool keep[8];
            int ej[8], kept = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                psel[j] = dpf[j] = 0.f;
                keep[j] = false;
                ej[j] = 0;
                if (j < k) {
                    ej[j] = min(max(__shfl(sm_idx, j, 16), 0), E - 1);
                    float mine = 0.f;
#pragma unroll
                    for (int i = 0; i < 4; ++i) mine = ej[j] == l + 16 * i ? v[i] : mine;
                    for (int o = 8; o > 0; o >>= 1) mine += __shfl_xor(mine, o);
                    psel[j] = mine;
                    const float dj = __shfl(sm_d, j, 16), uj = __shfl(sm_u, j, 16);
                    dpf[j] = __shfl(sm_inv, j, 16) >= 0 ? dj : 0.f;   // a capacity-dropped assignment carries no gradient from h'
                    if (cap.slots != nullptr) dpf[j] += capg_s[ej[j]];   // but it counts as assigned (capacity loss)
                    keep[j] = rate > 0.f ? !(uj < rate) : true;
                    kept += keep[j] ? 1 : 0;
                }
            }
            if (rate > 0.f) {
                if (kept == 0) keep[0] = true;
                float ssum = 0.f, dot = 0.f;
#pragma unroll
                for (int j = 0; j < 8; ++j) ssum += keep[j] ? psel[j] : 0.f;
#pragma unroll
                for (int j = 0; j < 8; ++j) dot += keep[j] ? dpf[j] * (psel[j] / ssum) : 0.f;
#pragma unroll
                for (int j = 0; j < 8; ++j) dpf[j] = keep[j] ? (dpf[j] - dot) / ssum : 0.f;
            }
            float csum = 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                dpf[j] = j < k ? dpf[j] * psel[j] * inv_tau : 0.f;
                csum += dpf[j];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = l + 16 * i;
                float t = -v[i] * csum;
#pragma unroll
                for (int j = 0; j < 8; ++j) t += j < k && e == ej[j] ? dpf[j] : 0.f;
                dgs[r * GST + e] = r < rows && e < E ? t : 0.f;   // slices past the end contribute nothing
            }
        }
        __syncthreads();
        // ---- dL/du of this wavefront's hidden tile (ReLU applied), and the weight gradients
        f32x16 du;
        float uv[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            du[i] = 0.f;
            uv[i] = u_r[acc_feature(i, 0) * UST];
        }
        if (AHEAD)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (8 * q >= E) break;
#pragma unroll
                for (int s = 0; s < 4; ++s) du = mfma_f32(dg_b[8 * q + s], dw[q][s], du);
            }
        for (int kb = AHEAD ? 32 : 0; kb < E; kb += 8) {
            float v[4];
            load_quad(Wr2 + (size_t)hidc * E + kb + 4 * g, E - kb - 4 * g, vec_e, v);
#pragma unroll
            for (int s = 0; s < 4; ++s) du = mfma_f32(dg_b[kb + s], v[s], du);
        }
        const int dx_t = wave % OTC, dx_k0 = wave / OTC * (kGbHidden / PARTS), dx_f = min(32 * dx_t + jj, own_n - 1);
        float bx[AHEAD ? 2 : 1][16];   // of dL/dh: the wavefront's 64 hidden units of Wr1's row dx_f
        static_assert(kGbHidden / PARTS == 64, "two batches");
        auto first_layer = [&](int kb, float (&b)[16]) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4];
                const T *at = (const T *)((const char *)(Wr1 + (size_t)own_c0 * Hr + kb + 8 * q) + ((unsigned)(dx_f * Hr + 4 * g) + here) * (unsigned)sizeof(T));
                if (AHEAD) Quad<T>::load(at, v);
                else load_quad(at, Hr - (kb + 8 * q + 4 * g), vec_hr, v);
#pragma unroll
                for (int s = 0; s < 4; ++s) b[4 * q + s] = v[s];
            }
        };
        // the expert path's rows of this thread's quad of dL/dh
        float4 xr[AHEAD ? 2 : 1];
        if (AHEAD) {
#pragma unroll
            for (int q = 0; q < 2; ++q) first_layer(dx_k0 + 32 * q, bx[q]);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int row = __shfl(sm_inv, min(j, k - 1), 16);
                xr[j] = *(const float4 *)(dxrow + (size_t)max(row, 0) * ds + own_c0 + 4 * sm_l);
            }
        }
        __syncthreads();   // everyone has taken its u: the region now takes dL/du
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int row = acc_feature(i, 0);   // and 4 g more, in the bases
            const float d = hok && uv[i] > 0.f ? du[i] : 0.f;
            ab1 += d;
            du_w[row] = d;
#pragma unroll
            for (int ot = 0; ot < OTC; ++ot) aW1[ot] = mfma_f32(xT_r[32 * ot * 36 + row], d, aW1[ot]);   // [feature][hidden unit]
            if (own == 0) {
                aW2[0] = mfma_f32(uv[i], dg_r[row * GST], aW2[0]);                                        // [hidden unit][expert]
                if (ET > 1) aW2[1] = mfma_f32(uv[i], dg_r[row * GST + 32], aW2[1]);
            }
        }
        if (own == 0 && tid < E)
            for (int r = 0; r < rows; ++r) ab2 += dgs[r * GST + tid];
        __syncthreads();
        {   // ---- dL/dh of the slices, own columns: router path ...
            f32x16 dx;
#pragma unroll
            for (int i = 0; i < 16; ++i) dx[i] = 0.f;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int kb = dx_k0 + 32 * q;
                if (kb >= Hr) break;
                if (!AHEAD) first_layer(kb, bx[0]);
                const float *du_b = us + (kb + 4 * g) * kGbT + jj;
#pragma unroll
                for (int s = 0; s < 16; ++s) dx = mfma_f32(du_b[(8 * (s >> 2) + (s & 3)) * kGbT], bx[AHEAD ? q : 0][s], dx);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) red_w[acc_feature(i, 0) * kGbT] = dx[i];
        }
        __syncthreads();
        // ... plus the expert-path rows of the k assignments
        if (AHEAD) {   // a quad per thread
            float v[4];
            const float *at = red + ((sm_l >> 3) * kGbRows + sm_r) * kGbT + (4 * sm_l & 31);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                v[c] = 0.f;
#pragma unroll
                for (int q = 0; q < PARTS; ++q) v[c] += at[q * OTC * kGbRows * kGbT + c];
            }
            auto add = [&](int j, float4 w) {
                const float wc[4] = {w.x, w.y, w.z, w.w};
                const bool has = j < k && __shfl(sm_inv, min(j, k - 1), 16) >= 0;
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = has ? v[c] + wc[c] : v[c];
            };
            add(0, xr[0]);
            add(1, xr[1]);
            for (int j = 2; j < k; ++j) add(j, *(const float4 *)(dxrow + (size_t)max(__shfl(sm_inv, j, 16), 0) * ds + own_c0 + 4 * sm_l));
            if (sm_r < rows) store_quad(dh + sm_n * ds + own_c0 + 4 * sm_l, v);
        } else
        for (int t = tid; t < rows * own_n; t += kGbThreads) {
            const int r = t / own_n, f = t - r * own_n;
            const long long n = n0 + r;
            float v = 0.f;
#pragma unroll
            for (int q = 0; q < PARTS; ++q) v += red[((q * OTC + (f >> 5)) * kGbRows + r) * kGbT + (f & 31)];
            for (int j = 0; j < k; ++j) {
                const int row = inv[n * k + j];
                if (row >= 0) v += dxrow[(size_t)row * ds + own_c0 + f];
            }
            Storage<T>::store(dh + n * ds + own_c0 + f, v);
        }
    }

    // ---- this block's slot: dWr1 [ds][Hr] | dWr2 [Hr][E] | dbr1 [Hr] | dbr2 [E]; the feature chunks write disjoint parts
    float *slot = part + (size_t)blockIdx.x * slot_floats;
    float *pWr1 = slot, *pWr2 = pWr1 + (size_t)ds * Hr, *pbr1 = pWr2 + (size_t)Hr * E, *pbr2 = pbr1 + Hr;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
#pragma unroll
        for (int ot = 0; ot < OTC; ++ot) {
            const int f = 32 * ot + acc_feature(i, g);
            if (hok && f < own_n) pWr1[(size_t)(own_c0 + f) * Hr + hid] = aW1[ot][i];
        }
        const int hr = wave * 32 + acc_feature(i, g);
        if (own == 0 && hr < Hr) {
            if (jj < E) pWr2[(size_t)hr * E + jj] = aW2[0][i];
            if (32 + jj < E) pWr2[(size_t)hr * E + 32 + jj] = aW2[1][i];
        }
    }
    ab1 += __shfl_xor(ab1, 32);
    if (own == 0 && g == 0 && hok) pbr1[hid] = ab1;
    if (own == 0 && tid < E) pbr2[tid] = ab2;
}

// ------------------------------------------------------------------------------------------------------ host
static int generic_col_tiles(int ds) { return ds <= 32 ? 1 : ds <= 64 ? 2 : 4; }   // columns per block of the expert kernel, in tiles

BackwardWeightsPlan backward_generic_plan(const slicemoe_config &c)
{
    BackwardWeightsPlan W;
    const long long Na = (long long)c.T * c.S * c.k;
    const int ds = c.d / c.S, cc = 32 * generic_col_tiles(ds);
    W.onepass = false;
    W.fused = true;
    W.groups = 1;
    W.step = kGbRows;
    // No position for beginning an expert: a slot costs a block a tenth of a unit, but whole units are handed out, and at the batches
    // this kernel runs at the extra positions often doubled a block's share.  8000 rows, 8 experts, 256 blocks: 254 units + 8
    // positions were two to a block (129 blocks at work, 53 us); one to a block 33 us, and 3 us more for twice the slots.
    W.overhead = 0;
    long long blocks = num_compute_units() / ((ds + cc - 1) / cc);
    const long long most = (Na + kGbRows - 1) / kGbRows + c.E - 1;   // units: an expert's rows begin one
    if (blocks > most) blocks = most;
    W.blocks = blocks < 1 ? 1 : (int)blocks;
    W.slots = W.reserve = (long long)W.blocks + c.E;
    return W;
}

static int generic_router_blocks(const slicemoe_config &c)   // at the most, of one chunk of columns
{
    const int ds = c.d / c.S, blocks = num_compute_units() / ((ds + kGrFeat - 1) / kGrFeat);
    return blocks < 1 ? 1 : blocks;
}
static int generic_router_units_per_block(const slicemoe_config &c)
{
    const long long units = ((long long)c.T * c.S + kGbRows - 1) / kGbRows, blocks = generic_router_blocks(c);
    const long long per = (units + blocks - 1) / blocks;
    return per < 1 ? 1 : (int)per;
}

long long backward_generic_router_slots(const slicemoe_config &c)
{
    const long long units = ((long long)c.T * c.S + kGbRows - 1) / kGbRows, per = generic_router_units_per_block(c);
    return (units + per - 1) / per;
}

long long backward_generic_router_slots_bound(const slicemoe_config &c)
{
    const long long units = ((long long)c.T * c.S + kGbRows - 1) / kGbRows, most = generic_router_blocks(c);
    return units < most ? units : most;
}

template <typename T> static bool quad_aligned(const void *p, int stride) { return stride % 4 == 0 && (uintptr_t)p % (4 * sizeof(T)) == 0; }

template <typename T, int OTC, bool AHEAD = false>
static hipError_t run_expert(const slicemoe_config &c, const void *h, const slicemoe_weights &w, const void *d_out, const float *pk,
                             const int32_t *offsets, const int32_t *perm, size_t slot_floats, float *dxrow, float *dpk, float *part, hipStream_t s)
{
    const int ds = c.d / c.S, cc = 32 * OTC;
    const bool vec_ds = quad_aligned<T>(w.W2, ds), vec_he = quad_aligned<T>(w.W1, c.He);
    if constexpr (OTC < 4 && !AHEAD)
        if (ds == cc && c.He % 32 == 0 && vec_ds && vec_he) return run_expert<T, OTC, true>(c, h, w, d_out, pk, offsets, perm, slot_floats, dxrow, dpk, part, s);
    const size_t lds = GenericExpertLds<OTC>::total * sizeof(float);
    auto kern = bwd_expert_generic_kernel<T, OTC, AHEAD>;
    const hipError_t e = grant_dynamic_lds((const void *)kern, lds);
    if (e != hipSuccess) return e;
    kern<<<dim3((unsigned)backward_generic_plan(c).blocks, (unsigned)((ds + cc - 1) / cc)), kGbThreads, lds, s>>>(
        (const T *)h, (const T *)d_out, pk, offsets, perm, ds, c.He, c.E, c.k, (const T *)w.W1, (const T *)w.b1, (const T *)w.W2,
        vec_ds, vec_he, dxrow, dpk, slot_floats, part);
    return hipGetLastError();
}

template <typename T>
static hipError_t run_generic(const slicemoe_config &c, const void *h, const slicemoe_weights &w, const void *d_out, const float *pk,
                              const int32_t *offsets, const int32_t *perm, size_t slot_floats, float *dxrow, float *dpk, float *part, hipStream_t s)
{
    switch (generic_col_tiles(c.d / c.S)) {
        case 1: return run_expert<T, 1>(c, h, w, d_out, pk, offsets, perm, slot_floats, dxrow, dpk, part, s);
        case 2: return run_expert<T, 2>(c, h, w, d_out, pk, offsets, perm, slot_floats, dxrow, dpk, part, s);
        default: return run_expert<T, 4>(c, h, w, d_out, pk, offsets, perm, slot_floats, dxrow, dpk, part, s);
    }
}

hipError_t launch_backward_expert_generic(const slicemoe_config &c, const void *h, const slicemoe_weights &w, const void *d_out,
                                          const float *pk, const int32_t *offsets, const int32_t *perm, size_t slot_floats, float *dxrow,
                                          float *dpk, float *part, hipStream_t s)
{
    return c.dtype == SLICEMOE_BF16 ? run_generic<bf16_t>(c, h, w, d_out, pk, offsets, perm, slot_floats, dxrow, dpk, part, s)
                                    : run_generic<float>(c, h, w, d_out, pk, offsets, perm, slot_floats, dxrow, dpk, part, s);
}

template <typename T>
static hipError_t run_router(const slicemoe_config &c, const void *h, const slicemoe_weights &w, const RouteVariant &v, const float *drop_u,
                             float rate, const int32_t *idx, const int32_t *inv, const float *dpk, const float *dxrow, void *d_h,
                             size_t slot_floats, float *part, hipStream_t s)
{
    const long long Ns = (long long)c.T * c.S;
    const int ds = c.d / c.S;
    const size_t lds = GenericRouterLds::total * sizeof(float);
    const bool ahead = c.Hr == kGbHidden && ds % kGrFeat == 0 && c.E % 8 == 0 && quad_aligned<T>(w.Wr1, c.Hr) && quad_aligned<T>(w.Wr2, c.E) &&
                       quad_aligned<T>(d_h, ds) && quad_aligned<float>(dxrow, ds);
    auto kern = ahead ? bwd_router_generic_kernel<T, true> : bwd_router_generic_kernel<T, false>;
    const hipError_t e = grant_dynamic_lds((const void *)kern, lds);
    if (e != hipSuccess) return e;
    kern<<<dim3((unsigned)backward_generic_router_slots(c), (unsigned)((ds + kGrFeat - 1) / kGrFeat)), kGbThreads, lds, s>>>(
        (const T *)h, Ns, ds, c.Hr, c.E, c.k, (const T *)w.Wr1, (const T *)w.br1, (const T *)w.Wr2, (const T *)w.br2,
        v.sigma > 0.f ? v.noise : nullptr, v.sigma, v.inv_tau, rate > 0.f ? drop_u : nullptr, rate, idx, inv, dpk,
        CapLoss{v.cap_slots, (short)v.cap_nslots, (short)v.cap_bits, v.cap_alpha}, dxrow, (T *)d_h,
        generic_router_units_per_block(c), quad_aligned<T>(w.Wr1, c.Hr), quad_aligned<T>(w.Wr2, c.E), part, slot_floats);
    return hipGetLastError();
}

hipError_t launch_backward_router_generic(const slicemoe_config &c, const void *h, const slicemoe_weights &w, const RouteVariant &v,
                                          const float *drop_u, float rate, const int32_t *idx, const int32_t *inv, const float *dpk,
                                          const float *dxrow, void *d_h, size_t slot_floats, float *part, hipStream_t s)
{
    return c.dtype == SLICEMOE_BF16 ? run_router<bf16_t>(c, h, w, v, drop_u, rate, idx, inv, dpk, dxrow, d_h, slot_floats, part, s)
                                    : run_router<float>(c, h, w, v, drop_u, rate, idx, inv, dpk, dxrow, d_h, slot_floats, part, s);
}

}  // namespace slicemoe
