// Generic router and expert kernels, fp32 arithmetic.  They take any shape within the library limits and either storage
// type, and serve the fp32 configuration and every shape the bf16 matrix-core kernels do not cover.
#include "mfma.h"
#include "output_role.h"
#include "wavefront.h"
#include <type_traits>

namespace slicemoe {

constexpr int kRB = 8;          // slices per block of the router
constexpr int kGenThreads = 256;
constexpr int kW2LdsBytes = 40 * 1024;   // Wr2 goes to LDS up to this size (fp32)
constexpr int kW2Rows = 1, kW2Columns = 2;   // ... a row of it per hidden unit, or a column per expert in quads (Hr a multiple of 4)

// Router of paper Section 3.1: g = ReLU(x Wr1 + br1) Wr2 + br2, softmax over E, top-k on the fp32 logits with ties to the
// lower expert index.  Every pre-activation and logit is one chain of fused multiply-adds in ascending input order (which
// experts win, and which hidden units are active, depends on no split of the sums), so the chains are what bounds it: one
// thread per hidden unit with eight slices side by side; one thread per logit, fed from LDS; 32 lanes per slice for the
// softmax and the selection.  2048 slices, ds = 64, Hr = 256, E = 8: 15.3 -> 11.5 us (logits from memory, softmax
// by one thread per slice before).  A logit's chain reads four hidden units of the slice and of its expert per LDS access (kW2Columns: Wr2
// by columns) where there was one, and the softmax and the selection go only as far across the lanes as there are experts: forward
// of 2048 slices 29.9 -> 29.1 us, of 16 384 72.8 -> 70.1, of 65 536 with E = 16 140 -> 131.
// HIST: leaves the block's chunk of the dispatch histogram behind.  An instance of its own: with a test of the table's address instead, the
// large batches that have no use for it took 5% longer (the router alone, E = 8, k = 2, 131 072 slices: 142 us against 133).
template <typename T, int W2LDS /* 0, kW2Rows or kW2Columns */, bool DROP, bool HIST>
__global__ __launch_bounds__(kGenThreads) void route_generic_kernel(
    const T *__restrict__ x, long long Ns, int ds, int Hr, int E, int k,
    const T *__restrict__ Wr1, const T *__restrict__ br1, const T *__restrict__ Wr2, const T *__restrict__ br2,
    const float *__restrict__ noise, float sigma, float inv_tau, const float *__restrict__ drop_u, float rate,
    int32_t *__restrict__ idx, float *__restrict__ pk, uint16_t *__restrict__ hist /* read only if HIST */, int hist_stride)
{
    __shared__ int counts[HIST ? 64 : 1];   // selections of this block per expert
    extern __shared__ __align__(16) float smem[];
    constexpr bool QUADS = W2LDS == kW2Columns;
    // row strides: whole quads of features; hidden units of neighbouring slices in different banks, in quads where Wr2's are
    const int dsp = (ds + 3) & ~3, ust = QUADS ? Hr + 4 : Hr + 1, wst = Hr + 4;
    float *xs = smem;                 // [kRB][dsp]
    float *us = xs + kRB * dsp;       // [kRB][ust]
    float *gs = us + kRB * ust;       // [kRB][E]
    float *w2s = gs + kRB * E;        // [Hr][E], or [E][wst] (W2LDS only)
    const int tid = threadIdx.x;
    if (HIST && tid < 64) counts[tid] = 0;
    const long long n0 = (long long)blockIdx.x * kRB;
    const int rows = (int)min((long long)kRB, Ns - n0);

    for (int i = tid; i < kRB * dsp; i += kGenThreads) {
        const int r = i / dsp, c = i - r * dsp;
        xs[i] = r < rows && c < ds ? Storage<T>::load(x + (n0 + r) * ds + c) : 0.f;
    }
    if (W2LDS)
        for (int i = tid; i < Hr * E; i += kGenThreads) {
            const float v = Storage<T>::load(Wr2 + i);
            if (QUADS) w2s[i % E * wst + i / E] = v;
            else w2s[i] = v;
        }
    __syncthreads();
    for (int j = tid; j < Hr; j += kGenThreads) {
        float acc[kRB];
        const float b = Storage<T>::load(br1 + j);
#pragma unroll
        for (int r = 0; r < kRB; ++r) acc[r] = b;
        const int ds4 = ds & ~3;
#pragma unroll 4
        for (int i = 0; i < ds4; i += 4) {
            float wv[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) wv[q] = Storage<T>::load(Wr1 + (size_t)(i + q) * Hr + j);
#pragma unroll
            for (int r = 0; r < kRB; ++r) {
                const float4 xq = *(const float4 *)(xs + r * dsp + i);
                acc[r] = fmaf(xq.x, wv[0], acc[r]);
                acc[r] = fmaf(xq.y, wv[1], acc[r]);
                acc[r] = fmaf(xq.z, wv[2], acc[r]);
                acc[r] = fmaf(xq.w, wv[3], acc[r]);
            }
        }
        for (int i = ds4; i < ds; ++i) {
            const float wv = Storage<T>::load(Wr1 + (size_t)i * Hr + j);
#pragma unroll
            for (int r = 0; r < kRB; ++r) acc[r] = fmaf(xs[r * dsp + i], wv, acc[r]);
        }
#pragma unroll
        for (int r = 0; r < kRB; ++r) us[r * ust + j] = fmaxf(acc[r], 0.f);
    }
    __syncthreads();
    for (int t = tid; t < kRB * E; t += kGenThreads) {
        const int r = t / E, e = t - r * E;
        float acc = Storage<T>::load(br2 + e);
        const float draw = noise != nullptr && r < rows ? noise[(n0 + r) * E + e] : 0.f;
        if (QUADS) {   // four hidden units of the slice and of the expert per load
#pragma unroll 8
            for (int j = 0; j < Hr; j += 4) {
                const float4 u = *(const float4 *)(us + r * ust + j), w = *(const float4 *)(w2s + e * wst + j);
                acc = fmaf(u.x, w.x, acc);
                acc = fmaf(u.y, w.y, acc);
                acc = fmaf(u.z, w.z, acc);
                acc = fmaf(u.w, w.w, acc);
            }
        } else
#pragma unroll 8
        for (int j = 0; j < Hr; ++j) acc = fmaf(us[r * ust + j], W2LDS ? w2s[j * E + e] : Storage<T>::load(Wr2 + (size_t)j * E + e), acc);
        // training-time logit noise (Section 5): before the selection and the softmax
        if (noise != nullptr && r < rows) acc = fmaf(sigma, draw, acc);
        gs[t] = acc;
    }
    __syncthreads();
    // 32 lanes per slice, experts l and l + 32
    const int r = tid >> 5, l = tid & 31;
    static_assert(kGenThreads == 32 * kRB, "32 lanes per slice");
    // the furthest lane that has an expert is less than twice as far (tests in unrolled loops: a loop from `far` down costs 64 experts 1 us)
    const int far = E > 16 ? 16 : E > 8 ? 8 : 4;
    float v0 = l < E ? gs[r * E + l] : -INFINITY, v1 = l + 32 < E ? gs[r * E + l + 32] : -INFINITY;
    float m = fmaxf(v0, v1);
#pragma unroll
    for (int o = 16; o > 0; o >>= 1)
        if (o <= far) m = fmaxf(m, __shfl_xor(m, o));
    float den = (l < E ? expf((v0 - m) * inv_tau) : 0.f) + (l + 32 < E ? expf((v1 - m) * inv_tau) : 0.f);   // softmax of g / tau (Appendix B)
#pragma unroll
    for (int o = 16; o > 0; o >>= 1)
        if (o <= far) den += __shfl_xor(den, o);
    const long long n = n0 + r;
    for (int j = 0; j < k; ++j) {
        float bv = v0;
        int best = l;
        if (v1 > bv) {
            bv = v1;
            best = l + 32;
        }
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) {
            if (o > far) continue;
            const float ov = __shfl_xor(bv, o);
            const int oe = __shfl_xor(best, o);
            if (ov > bv || (ov == bv && oe < best)) {
                bv = ov;
                best = oe;
            }
        }
        best = min(best, E - 1);   // only matters for logits that are not numbers
        if (l == 0 && r < rows) {
            idx[n * k + j] = best;
            pk[n * k + j] = expf((bv - m) * inv_tau) / den;
            if (HIST) atomicAdd(&counts[best], 1);
        }
        if (best == l) v0 = -INFINITY;
        if (best == l + 32) v1 = -INFINITY;
    }
    if (DROP && l == 0 && r < rows) drop_assignments(pk + n * k, drop_u + n * k, k, rate);   // (this lane has written them)
    if (HIST) {   // the block's chunk of the dispatch histogram
        __syncthreads();
        if (tid < E) {
            uint16_t *row = hist + (size_t)tid * hist_stride;
            row[blockIdx.x] = (uint16_t)counts[tid];
            if (blockIdx.x == gridDim.x - 1)   // the padding of a row reads as zero
                for (int c = (int)gridDim.x; c < hist_stride; ++c) row[c] = 0;
        }
    }
}

// Expert FFN of Section 3.1 on stacked rows with the Eq. 1 input weighting and the gather fused:
// y[r] = GELU((p x) W1[e] + b1[e]) W2[e] + b2[e], exact (erf) GELU.  y is fp32 for fp32 storage and
// fp16 for bf16 storage (same convention as the bf16 matrix-core kernels).
// A block of eight wavefronts takes 32 rows of one expert and runs both products on the fp32 matrix instruction
// (32 x 32 x 2, operands and sums fp32).  First product: a wavefront per 32-wide hidden tile, lane = hidden unit (its weights
// are coalesced rows of W1), registers = rows; the activations go to LDS; second product: lane = output feature, the
// hidden units of a tile split over several wavefronts when there are fewer output tiles than wavefronts.  Bound by the
// matrix instruction (64 cycles each) and the latency of the first weights; 4096 rows, ds = 64, He = 256: 75 ->
// 16 us (one thread per hidden unit reading its weights once per row before).  Takes what ffn_generic_ahead_kernel does not.
constexpr int kF32Threads = 512, kF32Waves = 8, kF32Rows = 32;
constexpr int kF32Feat = 128;              // features of the rows staged at a time
constexpr int kF32Hidden = 32 * kF32Waves;  // hidden units at a time
constexpr int kF32Batch = 16;               // weight loads in flight per lane

template <typename T, typename YT, int NO>
__global__ __launch_bounds__(kF32Threads) void ffn_generic_kernel(
    const T *__restrict__ x, const float *__restrict__ pk, const int32_t *__restrict__ offsets,
    const int32_t *__restrict__ perm, int ds, int He, int E, int k,
    const T *__restrict__ W1, const T *__restrict__ b1, const T *__restrict__ W2, const T *__restrict__ b2,
    YT *__restrict__ y)
{
    constexpr int XST = kF32Feat + 1, HST = kF32Hidden + 1;
    __shared__ float xs[kF32Rows * XST];                     // p x, features c0 .. of the rows
    __shared__ float hs[kF32Waves * kF32Rows * 33];          // activations [row][HST]; then partial outputs [wavefront][row][33]
    __shared__ int ns[kF32Rows];
    __shared__ float ps[kF32Rows];
    static_assert(kF32Rows * HST <= kF32Waves * kF32Rows * 33, "the activations fit");
    const int tid = threadIdx.x, lane = tid & 63, jj = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the block's expert and rows: units of 32 counted from each expert's first row
    const int off_lo = offsets[min(lane, E)], off_hi = offsets[min(lane + 1, E)];
    const int units = (off_hi - off_lo + kF32Rows - 1) / kF32Rows, first = wavefront_exclusive_scan(units, lane);
    const unsigned long long mine = __ballot((int)blockIdx.x >= first && (int)blockIdx.x < first + units);
    if (mine == 0) return;   // the grid is an upper bound; uniform
    const int e = __builtin_ctzll(mine);
    const int row0 = __builtin_amdgcn_readlane(off_lo, e) + ((int)blockIdx.x - __builtin_amdgcn_readlane(first, e)) * kF32Rows;
    const int nrows = min(kF32Rows, __builtin_amdgcn_readlane(off_hi, e) - row0);
    const T *w1 = W1 + (size_t)e * ds * He, *w2 = W2 + (size_t)e * He * ds;
    if (tid < kF32Rows) {
        const int a = perm[row0 + min(tid, nrows - 1)];
        ns[tid] = a / k;
        ps[tid] = tid < nrows ? pk[a] : 0.f;
    }
    __syncthreads();

    const int OT = (ds + 31) / 32;
    const OutputRole role = output_role(OT, kF32Waves, wave);
    const int parts = role.parts;
    f32x16 yacc[NO];
#pragma unroll
    for (int o = 0; o < NO; ++o)
#pragma unroll
        for (int i = 0; i < 16; ++i) yacc[o][i] = 0.f;
    for (int h0 = 0; h0 < He; h0 += kF32Hidden) {
        const int hid = h0 + wave * 32 + jj, hidc = min(hid, He - 1);
        f32x16 z;
        const float bias = Storage<T>::load(b1 + (size_t)e * He + hidc);
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = bias;
        for (int c0 = 0; c0 < ds; c0 += kF32Feat) {
            const int nf = min(kF32Feat, ds - c0), nf2 = (nf + 1) & ~1;
            if (h0 == 0 || ds > kF32Feat) {
                __syncthreads();   // everyone is done with the features before
                for (int i = tid; i < kF32Rows * kF32Feat; i += kF32Threads) {
                    const int r = i / kF32Feat, c = i % kF32Feat;
                    if (c < nf2) xs[r * XST + c] = c < nf ? ps[r] * Storage<T>::load(x + (size_t)ns[r] * ds + c0 + c) : 0.f;
                }
                __syncthreads();
            }
            const T *wp = w1 + (size_t)c0 * He + hidc;
            for (int k0 = 0; k0 < nf2; k0 += 2 * kF32Batch) {
                float b[kF32Batch];   // a batch of weights in flight at a time
#pragma unroll
                for (int s = 0; s < kF32Batch; ++s) b[s] = k0 + 2 * s + g < nf ? Storage<T>::load(wp + (size_t)(k0 + 2 * s + g) * He) : 0.f;
#pragma unroll
                for (int s = 0; s < kF32Batch; ++s)
                    if (k0 + 2 * s < nf2) z = __builtin_amdgcn_mfma_f32_32x32x2f32(xs[jj * XST + k0 + 2 * s + g], b[s], z, 0, 0, 0);
            }
        }
        __syncthreads();   // everyone is done with the activations before
#pragma unroll
        for (int i = 0; i < 16; ++i)
            hs[acc_feature(i, g) * HST + wave * 32 + jj] = hid < He ? 0.5f * z[i] * (1.f + erff(z[i] * 0.70710678118654752f)) : 0.f;
        __syncthreads();
        if (role.part < parts) {
            const int per = (kF32Hidden / parts + 1) & ~1, k0 = role.part * per, k1 = min(min(k0 + per, kF32Hidden), (He - h0 + 1) & ~1);
#pragma unroll
            for (int o = 0; o < NO; ++o) {
                const int f = 32 * (role.tile + kF32Waves * o) + jj, fc = min(f, ds - 1);
                if (role.has_tile(o)) {
                    for (int kb = k0; kb < k1; kb += 2 * kF32Batch) {
                        float b[kF32Batch];
#pragma unroll
                        for (int s = 0; s < kF32Batch; ++s)
                            b[s] = h0 + kb + 2 * s + g < He && kb + 2 * s < k1 ? Storage<T>::load(w2 + (size_t)(h0 + kb + 2 * s + g) * ds + fc) : 0.f;
#pragma unroll
                        for (int s = 0; s < kF32Batch; ++s)
                            if (kb + 2 * s < k1) yacc[o] = __builtin_amdgcn_mfma_f32_32x32x2f32(hs[jj * HST + kb + 2 * s + g], b[s], yacc[o], 0, 0, 0);
                    }
                }
            }
        }
    }
    if (parts == 1) {   // lane = feature, registers = rows
#pragma unroll
        for (int o = 0; o < NO; ++o) {
            const int f = 32 * (role.tile + kF32Waves * o) + jj;
            if (role.has_tile(o) && f < ds) {   // a wavefront without a tile has sums of nothing
                const float bias = Storage<T>::load(b2 + (size_t)e * ds + f);
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (acc_feature(i, g) < nrows) y[(size_t)(row0 + acc_feature(i, g)) * ds + f] = (YT)(yacc[o][i] + bias);
            }
        }
        return;
    }
    __syncthreads();
    if (role.part < parts)
#pragma unroll
        for (int i = 0; i < 16; ++i) hs[(wave * kF32Rows + acc_feature(i, g)) * 33 + jj] = yacc[0][i];
    __syncthreads();
    for (int t = tid; t < nrows * ds; t += kF32Threads) {
        const int r = t / ds, f = t - r * ds;
        float v = Storage<T>::load(b2 + (size_t)e * ds + f);
        for (int q = 0; q < parts; ++q) v += hs[((q * OT + (f >> 5)) * kF32Rows + r) * 33 + (f & 31)];
        y[(size_t)(row0 + r) * ds + f] = (YT)v;
    }
}

// The same for slices of exactly 32 OT columns and hidden widths of whole tiles, sums in the same order.  Such a layer's batches are
// mostly smaller than the chip, and then a block's time is the latency of its loads, one behind the other; without conditions they can
// all be requested ahead: the first product's weights with the rows, the second's before the activations, the output's bias with
// those.  Every wavefront reads the unit's indexes itself, so that there is no barrier between an index and its row.
// 8000 rows, ds = 64, He = 256: 18 -> 13 us; 32 768 rows (a forward pass): 108 -> 73 us, two blocks per compute unit instead of one
// (128 registers, 144 before; at ds = 64 that bound spills 8 to 10, four of them reloaded per 256 hidden units); ds = 32, He = 128, 131 072 rows: 289 -> 140.
template <typename T, typename YT, int OT>
__global__ __launch_bounds__(kF32Threads, 4) void ffn_generic_ahead_kernel(
    const T *__restrict__ x, const float *__restrict__ pk, const int32_t *__restrict__ offsets,
    const int32_t *__restrict__ perm, int He, int E, int k,
    const T *__restrict__ W1, const T *__restrict__ b1, const T *__restrict__ W2, const T *__restrict__ b2,
    YT *__restrict__ y)
{
    constexpr int DS = 32 * OT, XST = DS + 1, HST = kF32Hidden + 1, PARTS = kF32Waves / OT;
    constexpr int ROWS = kF32Threads / DS, STAGED = kF32Rows / ROWS;   // staging: a thread has one column of every ROWS-th row
    __shared__ float xs[kF32Rows * XST];                     // p x
    __shared__ float hs[kF32Waves * kF32Rows * 33];          // activations [row][HST]; then partial outputs [wavefront][row][33]
    const int tid = threadIdx.x, lane = tid & 63, jj = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int off_lo = offsets[min(lane, E)], off_hi = offsets[min(lane + 1, E)];
    const int units = (off_hi - off_lo + kF32Rows - 1) / kF32Rows, first = wavefront_exclusive_scan(units, lane);
    const unsigned long long mine = __ballot((int)blockIdx.x >= first && (int)blockIdx.x < first + units);
    if (mine == 0) return;   // the grid is an upper bound; uniform
    const int e = __builtin_ctzll(mine);
    const int row0 = __builtin_amdgcn_readlane(off_lo, e) + ((int)blockIdx.x - __builtin_amdgcn_readlane(first, e)) * kF32Rows;
    const int nrows = min(kF32Rows, __builtin_amdgcn_readlane(off_hi, e) - row0);
    const T *w1 = W1 + (size_t)e * DS * He, *w2 = W2 + (size_t)e * He * DS;
    const int a = perm[row0 + min(jj, nrows - 1)];
    const int st_c = tid % DS, st_r = tid / DS, tile = wave % OT, part = wave / OT;
    const float *xs_b = xs + jj * XST + g;
    float *hs_w = hs + 4 * g * HST + wave * 32 + jj;

    f32x16 yacc;
#pragma unroll
    for (int i = 0; i < 16; ++i) yacc[i] = 0.f;
    float ybias = 0.f;
    for (int h0 = 0; h0 < He; h0 += kF32Hidden) {
        const int hid = h0 + wave * 32 + jj, hidc = min(hid, He - 1);
        const float bias = Storage<T>::load(b1 + (size_t)e * He + hidc);
        float b[OT][16];
#pragma unroll
        for (int t = 0; t < OT; ++t)
#pragma unroll
            for (int s = 0; s < 16; ++s) b[t][s] = Storage<T>::load(w1 + (size_t)(32 * t + 2 * s) * He + (unsigned)(g * He + hidc));
        if (h0 == 0) {
            const int n = a / k;
            const float p = pk[a];
            float xv[STAGED];
#pragma unroll
            for (int q = 0; q < STAGED; ++q) xv[q] = Storage<T>::load(x + (size_t)__shfl(n, st_r + q * ROWS) * DS + st_c);
#pragma unroll
            for (int q = 0; q < STAGED; ++q) {
                const int r = st_r + q * ROWS;
                const float pr = __shfl(p, r);
                xs[r * XST + st_c] = r < nrows ? pr * xv[q] : 0.f;
            }
            __syncthreads();
        }
        f32x16 z;
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = bias;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < OT; ++t)
#pragma unroll
            for (int s = 0; s < 16; ++s) z = __builtin_amdgcn_mfma_f32_32x32x2f32(xs_b[32 * t + 2 * s], b[t][s], z, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < OT; ++t) {
            const int kb = min(part * DS + 32 * t, He - h0 - 32);   // (those past the end are not used)
#pragma unroll
            for (int s = 0; s < 16; ++s) b[t][s] = Storage<T>::load(w2 + (size_t)(h0 + kb + 2 * s) * DS + (unsigned)(g * DS + 32 * tile + jj));
        }
        if (h0 == 0) ybias = Storage<T>::load(b2 + (size_t)e * DS + st_c);
        __builtin_amdgcn_sched_barrier(0);
        if (h0 > 0) __syncthreads();   // everyone is done with the activations before
        if (h0 + 32 * wave < He)   // what lies past the end is not read
#pragma unroll
            for (int i = 0; i < 16; ++i) hs_w[acc_feature(i, 0) * HST] = 0.5f * z[i] * (1.f + erff(z[i] * 0.70710678118654752f));
        __syncthreads();
#pragma unroll
        for (int t = 0; t < OT; ++t) {
            const int kb = part * DS + 32 * t;
            if (kb >= He - h0) break;
            const float *hs_b = hs + jj * HST + kb + g;
#pragma unroll
            for (int s = 0; s < 16; ++s) yacc = __builtin_amdgcn_mfma_f32_32x32x2f32(hs_b[2 * s], b[t][s], yacc, 0, 0, 0);
        }
    }
    __syncthreads();
    float *out_w = hs + (wave * kF32Rows + 4 * g) * 33 + jj;
#pragma unroll
    for (int i = 0; i < 16; ++i) out_w[acc_feature(i, 0) * 33] = yacc[i];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < STAGED; ++q) {
        const int r = st_r + q * ROWS;
        const float *at = hs + ((st_c >> 5) * kF32Rows + r) * 33 + (st_c & 31);
        float v = ybias;
#pragma unroll
        for (int u = 0; u < PARTS; ++u) v += at[u * OT * kF32Rows * 33];
        if (r < nrows) y[(size_t)(row0 + r) * DS + st_c] = (YT)v;
    }
}

template <typename T>
static void run_route_generic(const slicemoe_config &c, const void *h, const slicemoe_weights &w, int32_t *idx, float *p, hipStream_t s,
                              const RouteVariant &v, uint16_t *hist, int hist_stride)
{
    const long long Ns = (long long)c.T * c.S;
    const int ds = c.d / c.S;
    const int blocks = (int)((Ns + kRB - 1) / kRB);
    const float *noise = v.sigma > 0.f ? v.noise : nullptr;
    const size_t rest = (size_t)kRB * (((ds + 3) & ~3) + c.E);                       // floats: slices and logits
    const size_t rows = rest + (size_t)kRB * (c.Hr + 1) + (size_t)c.Hr * c.E;        // with the hidden units and Wr2, in either layout
    const size_t quads = rest + (size_t)kRB * (c.Hr + 4) + (size_t)(c.Hr + 4) * c.E;
    const size_t limit = (64 * 1024 - (hist != nullptr ? 256 : 0)) / sizeof(float);   // (256 bytes: the counts)
    const bool small = sizeof(float) * (size_t)c.Hr * c.E <= kW2LdsBytes;
    const int place = small && c.Hr % 4 == 0 && quads <= limit ? kW2Columns : small && rows <= limit ? kW2Rows : 0;
    const size_t smem = sizeof(float) * (place == kW2Columns ? quads : place == kW2Rows ? rows : rest + (size_t)kRB * (c.Hr + 1));
    const bool drop = v.rate > 0.f;
    auto pick = [&](auto placed) {
        constexpr int W = decltype(placed)::value;
        return hist != nullptr ? (drop ? route_generic_kernel<T, W, true, true> : route_generic_kernel<T, W, false, true>)
                               : (drop ? route_generic_kernel<T, W, true, false> : route_generic_kernel<T, W, false, false>);
    };
    auto kern = place == kW2Columns ? pick(std::integral_constant<int, kW2Columns>())
                : place == kW2Rows  ? pick(std::integral_constant<int, kW2Rows>())
                                    : pick(std::integral_constant<int, 0>());
    kern<<<blocks, kGenThreads, smem, s>>>((const T *)h, Ns, ds, c.Hr, c.E, c.k, (const T *)w.Wr1, (const T *)w.br1, (const T *)w.Wr2,
                                           (const T *)w.br2, noise, v.sigma, v.inv_tau, v.drop_u, v.rate, idx, p, hist, hist_stride);
}

// A block's slices are a chunk of the dispatch histogram, in batches whose table is small enough for the scatter blocks to sum it: up to
// 16 384 slices with 16 experts, 4096 with 64; beyond, chunks of eight slices would make the scan longer than the histogram kernel that they
// save.  2048 slices, E = 8: forward 40.9 -> 38.5 us, the histogram's launch between router and scatter.
int route_generic_hist_chunk(const slicemoe_config &c)
{
    const long long Ns = (long long)c.T * c.S;
    return Ns > 0 && dispatch_geometry(Ns * c.k, c.E, kRB * c.k).fused ? kRB * c.k : 0;
}

hipError_t launch_route_generic(const slicemoe_config &c, const void *h, const slicemoe_weights &w,
                                int32_t *idx, float *p, hipStream_t s, const RouteVariant &v, int32_t *hist)
{
    const long long Ns = (long long)c.T * c.S;
    if (Ns == 0) return hipSuccess;
    int stride = 0;
    if (hist != nullptr) {
        if (route_generic_hist_chunk(c) == 0) return hipErrorInvalidValue;
        stride = dispatch_geometry(Ns * c.k, c.E, kRB * c.k).stride;
    }
    if (c.dtype == SLICEMOE_BF16) run_route_generic<bf16_t>(c, h, w, idx, p, s, v, (uint16_t *)hist, stride);
    else run_route_generic<float>(c, h, w, idx, p, s, v, (uint16_t *)hist, stride);
    return hipGetLastError();
}

template <typename T, typename YT>
static void run_ffn_generic(const slicemoe_config &c, const void *h, const float *p, const int32_t *offsets, const int32_t *perm,
                            const slicemoe_weights &w, void *y, hipStream_t s)
{
    const long long Na = (long long)c.T * c.S * c.k;
    const int ds = c.d / c.S, no = ((ds + 31) / 32 + kF32Waves - 1) / kF32Waves;   // output tiles per wavefront: ds < 2048
    const long long blocks = Na / kF32Rows + (Na < c.E ? Na : c.E);                 // at most one partial unit per expert
    auto kern = no <= 1 ? ffn_generic_kernel<T, YT, 1> : no <= 2 ? ffn_generic_kernel<T, YT, 2> : no <= 4 ? ffn_generic_kernel<T, YT, 4>
                                                                                               : ffn_generic_kernel<T, YT, 8>;
    if ((ds == 32 || ds == 64) && c.He % 32 == 0) {   // faster at every batch measured, one row to 131 072: 1.14 to 2.1 times (a forward pass)
        auto ahead = ds == 32 ? ffn_generic_ahead_kernel<T, YT, 1> : ffn_generic_ahead_kernel<T, YT, 2>;
        ahead<<<(unsigned)blocks, kF32Threads, 0, s>>>((const T *)h, p, offsets, perm, c.He, c.E, c.k, (const T *)w.W1, (const T *)w.b1,
                                                       (const T *)w.W2, (const T *)w.b2, (YT *)y);
        return;
    }
    kern<<<(unsigned)blocks, kF32Threads, 0, s>>>((const T *)h, p, offsets, perm, ds, c.He, c.E, c.k, (const T *)w.W1, (const T *)w.b1,
                                                  (const T *)w.W2, (const T *)w.b2, (YT *)y);
}

hipError_t launch_ffn_generic(const slicemoe_config &c, const void *h, const float *p,
                              const int32_t *offsets, const int32_t *perm, const slicemoe_weights &w,
                              void *y, hipStream_t s)
{
    if ((long long)c.T * c.S * c.k == 0) return hipSuccess;
    if (c.dtype == SLICEMOE_BF16) run_ffn_generic<bf16_t, _Float16>(c, h, p, offsets, perm, w, y, s);
    else run_ffn_generic<float, float>(c, h, p, offsets, perm, w, y, s);
    return hipGetLastError();
}

}  // namespace slicemoe
