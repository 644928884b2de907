// Matrix-core weight gradients of the experts, and for the narrow experts the whole expert backward in the same pass.
//
// The weight gradients contract over ROWS, which the forward's layout (a lane owns a row, see mfma.h) keeps on lanes.
// Swapping the operands of an MFMA transposes its result: with the row fragment as A and the weight fragment as B the
// accumulators of u = x W1 and da = dy W2^T come out as lane = hidden unit, registers = 16 of 32 rows.  There z, the
// activation a1 and p dz are formed, split into two bf16 terms (register pairs are row pairs: contraction slots), and
// dW2 += a1^T dy, dW1 += x^T (p dz) run on matrix instructions.  Their other operand, x and dy with lane = slice feature
// and slots = rows, comes out of the LDS by transposing reads (ds_read_b64_tr_b16), so no vector instruction is spent on it.
//
// A block's wavefronts own one hidden tile each and share the rows: units of 32 stacked rows of one expert are
// gathered into registers while the unit before is computed, and put into the LDS in front of the barrier.
//
// What bounds it: vector issue and its latency.  A hidden element takes about 30 vector instructions, two of them
// transcendental; measured on this chip a wavefront issues one every 4.7 cycles at best, waits 8.3 for the result of the
// one before (so the activation runs four elements side by side), and a SIMD with two wavefronts gets through one every
// 2.4.  Hence: no vector instructions for transposes (LDS), LDS reads in front of a run of vector instructions and the
// matrix instructions that use them behind it, the weight gradients half a unit behind the activation, barriers that do not
// wait for global memory, and the younger wavefront of a SIMD first for half of every unit.
//
// FUSE (experts whose hidden tiles fit one block: the benchmark shapes at width 64): the
// same pass also gives dL/dx and dL/dp of the rows, so that z and the activation are evaluated once instead of once per
// layout.  dx = W1 (p dz) contracts over the hidden units of ALL wavefronts, so the terms of p dz of a unit go through
// the LDS ([hidden][row], read back transposed) and during the next unit each wavefront multiplies its 16-row, 16-feature
// tile.  dL/dp = sum of dz u over the hidden units, which sit on lanes and wavefronts here: an exchange inside the
// wavefront that halves the number of values at every step, and one sum over the wavefronts.
//
// Measured, 524 288 rows, width 64, He = 256, 32 experts: rows kernel 172 us + weights kernel 283 us (both evaluating the
// activation, the latter without prefetch and with transposes on the matrix pipe) -> 254 us (236 at the least); the partial sums of
// the weight gradients fall from 140 MB in 1056 slots to 38 MB in 288 (their reduction 29-35 -> 12 us).  Unfused, alone on the
// chip, at width 128, He = 512: 2.78 -> 1.09 ms for 1 048 576 rows; width 96, He = 384: 228 -> 98 us for 131 056 rows.  (Widths 24
// and 48, and 96 where onepass_chosen says so: backward_expert_mfma.hip.)
//
// TERMS: bf16 terms of the activation and of p dz, backward_terms(DS).
#include "bwd_mfma.h"
#include "lds_rows.h"
#include "onepass_split.h"
#include "wavefront.h"

namespace slicemoe {

// p dz of a unit in the LDS: [term][hidden unit of the block][32 rows] bf16, the 8-byte quads of rows permuted inside a hidden unit's
// 64 bytes so that neither the writes (a lane per hidden unit) nor the transposing reads meet bank conflicts.
__device__ __forceinline__ int pdz_offset(int hidden, int quad)
{
    const int sw = ((hidden >> 2) & 1) | (((hidden >> 4) & 1) << 1) | (((hidden >> 3) & 1) << 2);
    return hidden * 64 + ((quad ^ sw) << 3);
}

constexpr int kUnit = kOnepassUnit;   // stacked rows a block works on at a time, as in the one-pass kernel

// Geometry of one instantiation.
template <int DS, int WAVES, int NBUF, bool WLDS, bool FUSE, int TERMS> struct WeightsTile {
    static constexpr int KS = SliceTiles<DS>::KS, OT = SliceTiles<DS>::OT, FT = DS / 16;
    static constexpr int THREADS = WAVES * 64;
    static constexpr int NBW = WAVES < 2 * OT ? WAVES : 2 * OT, TB = (2 * OT + NBW - 1) / NBW;   // wavefronts that add up db2, their shares
    static constexpr size_t rows_bytes = (size_t)2 * kUnit * LdsRows<DS>::STRIDE;                // x and dy of one unit
    static constexpr size_t pdz_bytes = (size_t)TERMS * WAVES * 32 * kUnit * 2;                  // p dz of one unit
    static constexpr size_t off_p = NBUF * rows_bytes;                                           // [NBUF][32] probabilities
    static constexpr size_t off_dp = off_p + NBUF * kUnit * 4;                                   // [2][WAVES][32] partial dL/dp
    static constexpr size_t off_db2 = off_dp + (FUSE ? 2 * WAVES * kUnit * 4 : 0);               // [2][32 OT] partial db2
    static constexpr size_t off_w = off_db2 + 2 * OT * 32 * 4;                                   // fragments of W1 and W2
    static constexpr size_t off_pdz = off_w + (WLDS ? (size_t)WAVES * KS * 2048 : 0);
    static constexpr size_t off_w1d = off_pdz + (FUSE ? 2 * pdz_bytes : 0);
    static constexpr size_t lds = off_w1d + (FUSE ? (size_t)FT * WAVES * 1024 : 0);
};

template <int DS, int WAVES, int NBUF, bool WLDS, bool FUSE, int TERMS, int MINWAVES>
__global__ __launch_bounds__(WAVES * 64, MINWAVES) void bwd_weights_kernel(
    const bf16_t *__restrict__ x, const bf16_t *__restrict__ dout, const float *__restrict__ pk,
    const int32_t *__restrict__ offsets, const int32_t *__restrict__ perm, const char *__restrict__ packed,
    size_t e_stride, size_t off_w2r, size_t off_w1d, size_t off_b1, int He, int E, int k, int blocks, int groups,
    size_t slot_floats, float *__restrict__ part, float *__restrict__ dxrow, float *__restrict__ dpk)
{
    typedef WeightsTile<DS, WAVES, NBUF, WLDS, FUSE, TERMS> G;
    typedef LdsRows<DS> LR;
    constexpr int KS = G::KS, OT = G::OT, THREADS = G::THREADS, P = LR::P, PW = LR::PW;
    constexpr int NX = 2 * kUnit * P / THREADS;   // 16-byte pieces (of x, then of dy) a thread moves per unit
    static_assert(!FUSE || NBUF == 2, "the fused kernel has one barrier per unit");
    static_assert(DS % 32 == 0 && NX * THREADS == 2 * kUnit * P, "whole tiles of features, a thread for every piece");
    extern __shared__ __align__(16) char lds[];

    const int tid = threadIdx.x, lane = tid & 63, jj = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int HT = He / 32;
    // consecutive blocks go to the eight XCDs in turn, each with its own L2: the groups of hidden tiles of a block's rows
    // take block ids that are equal modulo 8
    const int grp = (int)(blockIdx.x / 8) % groups;
    const int vb = (int)(blockIdx.x / (8 * groups)) * 8 + (int)(blockIdx.x % 8);
    if (vb >= blocks) return;
    const int ht = grp * WAVES + wave;
    const bool active = ht < HT;

    const int off_lo = offsets[min(lane, E)], off_hi = offsets[min(lane + 1, E)];
    const RowAxis A = row_axis(off_hi - off_lo, kUnit, 1, blocks, lane);
    const int c0 = vb * A.share, c1 = c0 + A.share;

    // ---- addresses that do not change
    int mrow[NX], mcol[NX], mdst[NX];   // row, feature and LDS offset of the pieces this thread moves
    const bf16_t *msrc[NX];
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const int q = tid + i * THREADS, half = q >= kUnit * P ? 1 : 0, r = q - half * kUnit * P;
        mrow[i] = r / P;
        mcol[i] = 8 * (r % P);
        msrc[i] = (half ? dout : x) + mcol[i];
        mdst[i] = half * kUnit * LR::STRIDE + LR::offset(mrow[i], r % P);
    }
    const int sw = LR::swizzle(jj);
    const int a_base = jj * LR::STRIDE + ((g ^ sw) << 4);   // piece 2 ks + g of row jj: a_base ^ (ks << 5)
    const int c16 = lane & 15, G4 = lane >> 4;
    const int trow = 4 * g + (c16 >> 2);                    // first row this lane points at in a transposing read
    const int t_base = trow * LR::STRIDE + (((2 * (G4 & 1) + ((lane & 3) >> 1)) ^ LR::swizzle(trow)) << 4) + 8 * (lane & 1);
    auto slice_of = [&](int a) { return divide_by_k(a, k); };

    if constexpr (PW > P) {   // the pieces past the slice width stay zero
        for (int t = tid; t < NBUF * 2 * kUnit * (PW - P); t += THREADS) {
            const int row = t / (PW - P), piece = P + t % (PW - P);
            *(uint4 *)(lds + (row / kUnit) * (kUnit * LR::STRIDE) + LR::offset(row % kUnit, piece)) = make_uint4(0, 0, 0, 0);
        }
    }

    if constexpr (FUSE) {   // hidden tiles past the last one: zeros in both operands of dL/dx, and nothing for dL/dp
        const uint4 zero = make_uint4(0, 0, 0, 0);
        if (!active) ((float *)(lds + G::off_dp))[((lane >> 5) * WAVES + wave) * kUnit + jj] = 0.f;
        if (!active)
            for (int t = lane; t < 2 * TERMS * 128; t += 64) *(uint4 *)(lds + G::off_pdz + ((t >> 7) * WAVES + wave) * 2048 + (t & 127) * 16) = zero;
        for (int t = tid; t < G::FT * (WAVES - HT) * 64; t += THREADS) {
            const int ft = t / ((WAVES - HT) * 64), r = t - ft * (WAVES - HT) * 64;
            *(uint4 *)(lds + G::off_w1d + (ft * WAVES + HT) * 1024 + r * 16) = zero;
        }
    }

    for (int e = 0; e < E; ++e) {
        const int first = __builtin_amdgcn_readlane(A.first, e), steps = __builtin_amdgcn_readlane(A.steps, e);
        if (first >= c1) break;
        const int s_lo = max(0, c0 - first - 1), s_hi = min(steps, c1 - first - 1);
        if (s_hi <= s_lo) continue;
        const int row0 = __builtin_amdgcn_readlane(off_lo, e) + s_lo * kUnit;   // rows below count from here
        const int nrows = min(__builtin_amdgcn_readlane(off_hi, e) - row0, (s_hi - s_lo) * kUnit);
        const int32_t *ids = perm + row0;
        const char *ew = packed + (size_t)e * e_stride;

        __syncthreads();   // everyone is done with the LDS of the segment before
        // ---- this expert's weights
        bf16x8 w1r[WLDS ? 1 : KS], w2q[WLDS ? 1 : KS];
        const int htc = active ? ht : 0;
        if constexpr (WLDS) {
            const int nt = min(WAVES, HT - grp * WAVES);
            stage_bytes(ew + (size_t)grp * WAVES * KS * 1024, lds + G::off_w, (size_t)nt * KS * 1024, tid, THREADS);
            stage_bytes(ew + off_w2r + (size_t)grp * WAVES * KS * 1024, lds + G::off_w + (size_t)WAVES * KS * 1024, (size_t)nt * KS * 1024, tid,
                        THREADS);
        } else {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                w1r[ks] = __builtin_bit_cast(bf16x8, ((const uint4 *)ew)[(htc * KS + ks) * 64 + lane]);
                w2q[ks] = __builtin_bit_cast(bf16x8, ((const uint4 *)(ew + off_w2r))[(htc * KS + ks) * 64 + lane]);
            }
        }
        if constexpr (FUSE)
            for (int ft = 0; ft < G::FT; ++ft)
                stage_bytes(ew + off_w1d + (size_t)ft * HT * 1024, lds + G::off_w1d + ft * WAVES * 1024, (size_t)HT * 1024, tid, THREADS);
        const float bias = ((const float *)(ew + off_b1))[htc * 32 + jj];
        auto w1_frag = [&](int ks) {
            return WLDS ? __builtin_bit_cast(bf16x8, ((const uint4 *)(lds + G::off_w))[(wave * KS + ks) * 64 + lane]) : w1r[WLDS ? 0 : ks];
        };
        auto w2_frag = [&](int ks) {
            return WLDS ? __builtin_bit_cast(bf16x8, ((const uint4 *)(lds + G::off_w))[((WAVES + wave) * KS + ks) * 64 + lane]) : w2q[WLDS ? 0 : ks];
        };

        f32x16 aW1[OT], aW2[OT];
        float ab1 = 0.f, ab2[G::TB];
#pragma unroll
        for (int t = 0; t < G::TB; ++t) ab2[t] = 0.f;
#pragma unroll
        for (int ot = 0; ot < OT; ++ot)
#pragma unroll
            for (int i = 0; i < 16; ++i) aW1[ot][i] = aW2[ot][i] = 0.f;

        // ---- gather of a unit: assignment ids two units ahead, rows one unit ahead.  The slices are worked out from the ids
        // in front of a unit's stores of dL/dx, which would otherwise have to complete before the ids can be used.
        int an[NX], ao_next = 0, ao_load = 0, ao = 0;
        uint4 mv[NX];
        float p_next = 0.f;
        auto load_ids = [&](int r0) {
#pragma unroll
            for (int i = 0; i < NX; ++i) an[i] = ids[(unsigned)min(r0 + mrow[i], nrows - 1)];
            if (tid < kUnit) ao_next = ids[(unsigned)min(r0 + tid, nrows - 1)];
        };
        auto find_slices = [&]() {
            // (Both waited for here on every path: left to their uses, the first wavefront waits for them behind the unit's stores.)
#pragma unroll
            for (int i = 0; i < NX; ++i) asm volatile("" : "+v"(an[i]));
            asm volatile("" : "+v"(ao_next));
#pragma unroll
            for (int i = 0; i < NX; ++i) an[i] = slice_of(an[i]);
        };
        auto load_rows = [&]() {
#pragma unroll
            for (int i = 0; i < NX; ++i) mv[i] = *(const uint4 *)(msrc[i] + (size_t)an[i] * DS);
            if (tid < kUnit) {
                ao_load = ao_next;
                p_next = pk[ao_next];
            }
        };
        auto store_rows = [&](int r0, int buf) {   // rows past the end: dy and p are zero, so they add nothing
#pragma unroll
            for (int i = 0; i < NX; ++i) {
                const int q = tid + i * THREADS;
                *(uint4 *)(lds + buf * G::rows_bytes + mdst[i]) = q < kUnit * P || r0 + mrow[i] < nrows ? mv[i] : make_uint4(0, 0, 0, 0);
            }
            if (tid < kUnit) {
                ao = ao_load;
                ((float *)(lds + G::off_p))[buf * kUnit + tid] = r0 + tid < nrows ? p_next : 0.f;
            }
        };
        load_ids(0);
        find_slices();
        load_rows();
        store_rows(0, 0);
        load_ids(kUnit);   // (past the end: the last row's)
        find_slices();
        __syncthreads();

        // ---- dL/dx of the unit before (FUSE): 16-row, 16-feature tiles, lane = row c16 of the tile, dealt out to the
        // wavefronts; one 32-wide contraction step `kk` is one hidden tile (zeros past the last one: no branch).  For the
        // first unit of a segment it works on what the buffers hold, and nothing of it is stored.
        constexpr int NT = FUSE ? (2 * G::FT + WAVES - 1) / WAVES : 1;
        f32x4 dx[NT];
        struct DxFrags {
            bf16x8 w[NT], b[NT][TERMS];
        };
        auto dx_load = [&](DxFrags &f, int kk, int buf) {
            const char *pz = lds + G::off_pdz + buf * G::pdz_bytes;
            const int h0 = 8 * G4 + (c16 >> 2);
            const uint4 *w1d = (const uint4 *)(lds + G::off_w1d);
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const int tile = wave + i * WAVES, rt = tile & 1;
                const int ft = NT * WAVES == 2 * G::FT ? tile >> 1 : min(tile >> 1, G::FT - 1);   // a tile too many is not stored
                const char *b0 = pz + pdz_offset(h0, 4 * rt + (c16 & 3)) + kk * 2048;
                const char *b1 = pz + pdz_offset(h0 + 4, 4 * rt + (c16 & 3)) + kk * 2048;
                f.w[i] = __builtin_bit_cast(bf16x8, w1d[(ft * WAVES + kk) * 64 + lane]);
#pragma unroll
                for (int t = 0; t < TERMS; ++t) f.b[i][t] = read_transposed(as_lds(b0 + t * WAVES * 2048), as_lds(b1 + t * WAVES * 2048));
            }
        };
        auto dx_mma = [&](const DxFrags &f) {
#pragma unroll
            for (int t = TERMS - 1; t >= 0; --t)   // small terms first
#pragma unroll
                for (int i = 0; i < NT; ++i) dx[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.w[i], f.b[i][t], dx[i], 0, 0, 0);
        };
        auto dx_all = [&](int buf) {
            for (int kk = 0; kk < WAVES; ++kk) {
                DxFrags f;
                dx_load(f, kk, buf);
                dx_mma(f);
            }
        };
        auto dx_begin = [&]() {
#pragma unroll
            for (int i = 0; i < NT; ++i) dx[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        };
        float *dxs = FUSE ? dxrow + (size_t)row0 * DS : nullptr;
        auto dx_end = [&](int r0, int buf, int a) {   // stores the rows r0 ..; a: this thread's assignment
            // (Opaque copies: an address stepped from unit to unit would be a register reloaded from scratch in front of the loop, and a wait for
            // that reload at the end of every unit is one for the unit's stores.)
            int jo = c16, go = G4;
            asm volatile("" : "+v"(jo), "+v"(go));
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const int tile = wave + i * WAVES, row = r0 + 16 * (tile & 1) + jo, col = 16 * (tile >> 1) + 4 * go;
                if ((tile >> 1) < G::FT && row < nrows)   // (bytes: a segment's dL/dx is below 4 GB)
                    *(f32x4 *)((char *)dxs + ((unsigned)row * (4u * DS) + 4u * (unsigned)col)) = 0.5f * dx[i];
            }
            if (tid < kUnit && r0 + tid < nrows) {
                const float *dps = (const float *)(lds + G::off_dp) + buf * WAVES * kUnit + tid;
                float v[WAVES], t = 0.f;
#pragma unroll
                for (int w = 0; w < WAVES; ++w) v[w] = dps[w * kUnit];
#pragma unroll
                for (int w = 0; w < WAVES; ++w) t += v[w];
                dpk[a] = 0.5f * t;
            }
        };

        int buf = 0, a_prev = 0;
        for (int r0 = 0; r0 < nrows; r0 += kUnit) {
            const bool more = r0 + kUnit < nrows;
            const int a_cur = ao;
            if (more) {
                load_rows();
                load_ids(r0 + 2 * kUnit);
            }
            char *xs = lds + (NBUF == 2 ? buf : 0) * G::rows_bytes, *gs = xs + kUnit * LR::STRIDE;
            const float *ps = (const float *)(lds + G::off_p) + (NBUF == 2 ? buf : 0) * kUnit;
            // the transposed fragment i (rows 16 (i & 1) .., features 32 (i >> 1) ..) of x or dy
            auto transposed = [&](const char *rows, int i) {
                const int at = 16 * (i & 1) * LR::STRIDE, col = t_base ^ ((i >> 1) << 6);
                return read_transposed(as_lds(rows + at + col), as_lds(rows + at + 8 * LR::STRIDE + (col ^ 32)));
            };
            if constexpr (FUSE) dx_begin();
            if (active) {
                // lane = hidden unit jj of this tile, register i = row acc_feature(i, g) of the unit
                f32x16 u, da;
#pragma unroll
                for (int i = 0; i < 16; ++i) u[i] = da[i] = 0.f;
                constexpr int KH = KS <= 4 ? KS : KS % 4 == 0 ? 4 : 3;   // fragments requested together
                static_assert(KS % KH == 0, "whole groups of K-steps");
#pragma unroll
                for (int k0 = 0; k0 < KS; k0 += KH) {
                    bf16x8 xa[KH], ga[KH];
#pragma unroll
                    for (int ks = 0; ks < KH; ++ks) {
                        const int at = a_base ^ ((k0 + ks) << 5);
                        xa[ks] = *(const bf16x8 *)(xs + at);
                        ga[ks] = *(const bf16x8 *)(gs + at);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int ks = 0; ks < KH; ++ks) {
                        u = mfma_bf16(xa[ks], w1_frag(k0 + ks), u);
                        da = mfma_bf16(ga[ks], w2_frag(k0 + ks), da);
                    }
                }
                // The weight gradients run half a unit (16 rows, one K-step) behind the activation, and dL/dx of the unit
                // before runs beside it, so that the matrix pipe works while the vector instructions of the next half are
                // issued.  A quad of registers is two runs of vector instructions (about 60 each); in front of each run stand
                // the LDS reads, behind it the matrix instructions that use them: the reads' latency is covered by the run.
                uint32_t a1[2][TERMS][4], pdz[2][TERMS][4];   // by half of the unit; terms, the largest first
                bf16x8 gt, xt;
                auto second_load = [&](int half, int ot) {
                    gt = transposed(gs, 2 * ot + half);
                    xt = transposed(xs, 2 * ot + half);
                };
                auto second_mma = [&](int half, int ot) {   // small terms first
                    auto frag = [](const uint32_t (&v)[4]) { return __builtin_bit_cast(bf16x8, make_uint4(v[0], v[1], v[2], v[3])); };
#pragma unroll
                    for (int t = TERMS - 1; t >= 0; --t) {
                        aW2[ot] = mfma_bf16(frag(a1[half][t]), gt, aW2[ot]);    // [hidden unit][slice feature]: lane = feature
                        aW1[ot] = mfma_bf16(xt, frag(pdz[half][t]), aW1[ot]);   // [slice feature][hidden unit]: lane = hidden unit
                    }
                };
                float du[8];   // dz u, summed over the hidden units below
                // Of two wavefronts on a SIMD the older is served first, and would then wait at the barrier for the younger
                // working alone; so the younger goes first in the first half of the unit.
                if (wave >= WAVES / 2) __builtin_amdgcn_s_setprio(1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int half = 0; half < 2; ++half)
#pragma unroll
                    for (int qd = 0; qd < 2; ++qd) {   // registers 8 half + 4 qd ..: rows 8 q + 4 g ..
                        const int q = 2 * half + qd;
                        if (q == 2) __builtin_amdgcn_s_setprio(0);
                        // output tiles of the second stage behind each run (half 1 only): [o0, o1) and [o1, o2), the
                        // first of each with its reads in front of the run
                        const int o0 = qd == 0 ? 0 : OT / 2, o2 = qd == 0 ? OT / 2 : OT, o1 = (o0 + o2 + 1) / 2;
                        const f32x4 pv = *(const f32x4 *)(ps + 8 * q + 4 * g);
                        DxFrags fr;
                        if (FUSE && 2 * q < WAVES) dx_load(fr, 2 * q, buf ^ 1);
                        if (half == 1 && o0 < o1) second_load(0, o0);
                        __builtin_amdgcn_sched_barrier(0);
                        float z[4], dz[4], act[4], slope[4], pd[4];
#pragma unroll
                        for (int c = 0; c < 4; ++c) z[c] = fmaf(pv[c], u[4 * q + c], bias);
                        twice_gelu4(z, act, slope);
                        __builtin_amdgcn_sched_barrier(0);
                        if (FUSE && 2 * q < WAVES) dx_mma(fr);
                        if (half == 1) {
#pragma unroll
                            for (int ot = 0; ot < OT; ++ot) {
                                if (ot > o0 && ot < o1) second_load(0, ot);
                                if (ot >= o0 && ot < o1) second_mma(0, ot);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        if (FUSE && 2 * q + 1 < WAVES) dx_load(fr, 2 * q + 1, buf ^ 1);
                        if (half == 1 && o1 < o2) second_load(0, o1);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int c = 0; c < 4; ++c) dz[c] = da[4 * q + c] * slope[c];   // twice dL/dz
#pragma unroll
                        for (int c = 0; c < 4; ++c) pd[c] = pv[c] * dz[c];
                        split_terms<TERMS>(act, a1[half], 2 * qd);
                        split_terms<TERMS>(pd, pdz[half], 2 * qd);
                        ab1 += (dz[0] + dz[1]) + (dz[2] + dz[3]);
                        if constexpr (FUSE) {
#pragma unroll
                            for (int c = 0; c < 4; ++c)
                                du[4 * qd + c] = half == 0 ? dz[c] * u[4 * q + c] : sum_over_row_pair(du[4 * qd + c], dz[c] * u[4 * q + c]);
                            char *dst = lds + G::off_pdz + buf * G::pdz_bytes + pdz_offset(wave * 32 + jj, 2 * q + g);
#pragma unroll
                            for (int t = 0; t < TERMS; ++t) *(uint2 *)(dst + t * WAVES * 2048) = make_uint2(pdz[half][t][2 * qd], pdz[half][t][2 * qd + 1]);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        if (FUSE && 2 * q + 1 < WAVES) dx_mma(fr);
                        if (half == 1) {
#pragma unroll
                            for (int ot = 0; ot < OT; ++ot) {
                                if (ot > o1 && ot < o2) second_load(0, ot);
                                if (ot >= o1 && ot < o2) second_mma(0, ot);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                second_load(1, 0);
                if constexpr (FUSE) {   // dL/dp: this tile's hidden units; every fourth lane ends up with the sums of two rows
                    sum_over_hidden(du);
                    if ((lane & 3) == 0)
                        *(float2 *)((float *)(lds + G::off_dp) + (buf * WAVES + wave) * kUnit + hidden_sum_row(lane)) = make_float2(du[0], du[1]);
                }
#pragma unroll
                for (int ot = 0; ot < OT; ++ot) {
                    if (ot > 0) second_load(1, ot);
                    second_mma(1, ot);
                }
            } else if (FUSE) {
                dx_all(buf ^ 1);
            }
            if (grp == 0 && wave < G::NBW) {   // db2: sums of dy over the rows, the fragments dealt out to the wavefronts
#pragma unroll
                for (int t = 0; t < G::TB; ++t)
                    if (wave + t * G::NBW < 2 * OT) ab2[t] += fragment_sum(transposed(gs, wave + t * G::NBW));
            }
            if (NBUF == 2 && more) store_rows(r0 + kUnit, buf ^ 1);
            find_slices();
            if (FUSE && r0 > 0) dx_end(r0 - kUnit, buf ^ 1, a_prev);
            lds_barrier();
            if (NBUF == 1) {
                if (more) store_rows(r0 + kUnit, 0);
                lds_barrier();
            }
            a_prev = a_cur;
            buf ^= 1;
        }
        if constexpr (FUSE) {   // the last unit's dL/dx
            dx_begin();
            dx_all(buf ^ 1);
            dx_end((s_hi - s_lo - 1) * kUnit, buf ^ 1, a_prev);
        }

        // ---- this segment's slot: dW1 [ds][He] | dW2 [He][ds] | db1 [He] | db2 [ds]
        int he = He, jo = jj, go = g;   // opaque copies: the store addresses are made here, not kept in registers through the loop above
        asm volatile("" : "+s"(he), "+v"(jo), "+v"(go));
        float *slot = part + (size_t)(vb + e) * slot_floats;
        float *pW1 = slot, *pW2 = pW1 + (size_t)DS * he, *pb1 = pW2 + (size_t)he * DS, *pb2 = pb1 + he;
        float *red = (float *)(lds + G::off_db2);
        __syncthreads();
        if (active) {
#pragma unroll
            for (int ot = 0; ot < OT; ++ot)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int f = 32 * ot + acc_feature(i, go);
                    pW1[(size_t)f * he + 32 * ht + jo] = 0.5f * aW1[ot][i];
                    pW2[(size_t)(32 * ht + acc_feature(i, go)) * DS + 32 * ot + jo] = 0.5f * aW2[ot][i];
                }
            ab1 += __shfl_xor(ab1, 32);   // the two lane groups hold different rows of the same hidden unit
            if (go == 0) pb1[32 * ht + jo] = 0.5f * ab1;
        }
        if (grp == 0 && wave < G::NBW) {
#pragma unroll
            for (int t = 0; t < G::TB; ++t) {
                const int i = wave + t * G::NBW;   // rows 16 (i & 1) .. of every unit, features 32 (i >> 1) ..
                const float v = ab2[t] + __shfl_xor(ab2[t], 32);
                if (i < 2 * OT && g == 0) red[(i & 1) * OT * 32 + 32 * (i >> 1) + jj] = v;
            }
        }
        __syncthreads();
        if (grp == 0)
            for (int f = tid; f < DS; f += THREADS) pb2[f] = red[f] + red[OT * 32 + f];
    }
}

// ------------------------------------------------------------------------------------------------------ host
// Instantiations by slice width: wavefronts per block, row buffers, weights in LDS, fused, terms, wavefronts per SIMD the
// registers allow.
//   64            fused where the expert's hidden tiles fit one block (He <= 256): see the header
//   96, 128       64 accumulators and weights per hidden tile leave no registers for the fragments (LDS) or for dL/dx
//   192           192 accumulators: one wavefront per SIMD
struct WeightsConfig {
    int waves, per_cu;
};
static WeightsConfig weights_config(int ds, int He)
{
    if (ds == 64) return {He <= 128 ? 4 : 8, 1};
    if (ds == 96) return {4, 2};
    if (ds == 128) return {8, 1};
    return {4, 1};
}

static BackwardWeightsPlan weights_kernel_plan(const slicemoe_config &c)
{
    BackwardWeightsPlan W;
    const WeightsConfig C = weights_config(c.d / c.S, c.He);
    const int HT = c.He / 32;
    const long long Na = (long long)c.T * c.S * c.k;
    W.onepass = false;
    W.fused = weights_fused(c.d / c.S, c.He);
    W.step = kUnit;
    W.overhead = 1;
    W.groups = (HT + C.waves - 1) / C.waves;
    long long blocks = (long long)num_compute_units() * C.per_cu / W.groups;
    const long long most = (Na + kUnit - 1) / kUnit;
    if (blocks > most) blocks = most;
    W.blocks = blocks < 1 ? 1 : (int)blocks;
    W.slots = W.reserve = (long long)W.blocks + c.E;
    return W;
}

BackwardWeightsPlan backward_weights_plan(const slicemoe_config &c)
{
    const int ds = c.d / c.S;
    if (!onepass_depends_on_batch(ds, c.He)) return onepass_in_every_batch(ds, c.He) ? backward_expert_plan(c) : weights_kernel_plan(c);
    const long long units = ((long long)c.T * c.S * c.k + kUnit - 1) / kUnit;
    BackwardWeightsPlan one = backward_expert_plan(c), two = weights_kernel_plan(c);
    one.reserve = two.reserve = one.reserve > two.reserve ? one.reserve : two.reserve;
    return onepass_chosen(ds, c.He, c.E, units, num_compute_units()) ? one : two;
}

template <int DS, int WAVES, int NBUF, bool WLDS, bool FUSE, int TERMS, int MINWAVES>
static hipError_t run_weights(const slicemoe_config &c, const BackwardWeightsPlan &W, const BwdPacked &L, const void *h, const void *d_out,
                              const float *pk, const int32_t *offsets, const int32_t *perm, const char *packed, size_t slot_floats,
                              float *part, float *dxrow, float *dpk, hipStream_t s)
{
    typedef WeightsTile<DS, WAVES, NBUF, WLDS, FUSE, TERMS> G;
    if (W.fused != FUSE || W.groups != (c.He / 32 + WAVES - 1) / WAVES) return hipErrorInvalidValue;
    auto kern = bwd_weights_kernel<DS, WAVES, NBUF, WLDS, FUSE, TERMS, MINWAVES>;
    const hipError_t e = grant_dynamic_lds((const void *)kern, G::lds);
    if (e != hipSuccess) return e;
    kern<<<(unsigned)((W.blocks + 7) / 8 * 8 * W.groups), WAVES * 64, G::lds, s>>>(
        (const bf16_t *)h, (const bf16_t *)d_out, pk, offsets, perm, packed, L.stride, L.w2r, L.w1d, L.b1, c.He, c.E, c.k, W.blocks,
        W.groups, slot_floats, part, dxrow, dpk);
    return hipGetLastError();
}

hipError_t launch_backward_weights(const slicemoe_config &c, const BackwardWeightsPlan &W, const BwdPacked &L, const void *h, const void *d_out, const float *pk,
                                   const int32_t *offsets, const int32_t *perm, const char *packed, size_t slot_floats, float *part,
                                   float *dxrow, float *dpk, hipStream_t s)
{
    const int ds = c.d / c.S, waves = weights_config(ds, c.He).waves;
#define SLICEMOE_WEIGHTS(DS, WAVES, NBUF, WLDS, FUSE, MINW)                                                                        \
    if (ds == DS && waves == WAVES && W.fused == FUSE)                                                                              \
        return run_weights<DS, WAVES, NBUF, WLDS, FUSE, backward_terms(DS), MINW>(c, W, L, h, d_out, pk, offsets, perm, packed,      \
                                                                                  slot_floats, part, dxrow, dpk, s);
    SLICEMOE_WEIGHTS(64, 4, 2, false, true, 2)
    SLICEMOE_WEIGHTS(64, 8, 2, false, true, 2)
    SLICEMOE_WEIGHTS(64, 8, 2, false, false, 2)
    SLICEMOE_WEIGHTS(96, 4, 1, true, false, 2)
    SLICEMOE_WEIGHTS(128, 8, 1, true, false, 2)
    SLICEMOE_WEIGHTS(192, 4, 1, true, false, 1)
#undef SLICEMOE_WEIGHTS
    return hipErrorInvalidValue;
}

}  // namespace slicemoe
