// Matrix-core backward of the experts in one pass over the rows, for the paper's narrow slices (widths 24, 48 and 96): weight
// gradients, dL/dx and dL/dp from one evaluation of the activation.
//
// The weight gradients contract over ROWS, which the forward's layout (a lane owns a row, see mfma.h) keeps on lanes.
// Swapping the operands of an MFMA transposes its result: with the row fragment as A and the weight fragment as B the
// accumulators of u = x W1 and da = dy W2^T come out as lane = hidden unit, registers = rows.  There z, the
// activation a1 and p dz are formed, split into bf16 terms (register pairs are row pairs: contraction slots), and
// dW2 += a1^T dy, dW1 += x^T (p dz) run on matrix instructions.  Their other operand, x and dy with lane = slice feature
// and slots = rows, comes out of the LDS by transposing reads (ds_read_b64_tr_b16).  dx = W1 (p dz) contracts over the
// hidden units of ALL wavefronts, so the terms of p dz of a 32-row unit go through the LDS, and while the next unit is
// worked on the block's wavefronts multiply 16-row, 16-feature tiles of it.  dL/dp = sum of dz u over the hidden units, which
// sit on lanes and wavefronts here: an exchange inside the wavefront that halves the number of values at every step, and one
// sum over the wavefronts.
//
// Work split.  A wavefront owns SIXTEEN hidden units (v_mfma_f32_16x16x32_bf16 throughout), so that the sums of its weight gradients
// take ds / 2 registers and three wavefronts fit a SIMD (168 registers each; four of 128 at width 24): a wavefront alone issues an instruction every 5 to 6
// cycles, two and more get through one every 2.6 (fp32 multiply-add) to 4.6 (conversions, shifts).  Experts with more hidden
// units than a block has wavefronts for go through the same rows again, pass after pass: dL/dx and dL/dp of the passes before are
// read back by the thread that wrote them and added to.
//
// What bounds it: vector issue (about 300 instructions per wavefront and unit) and the phases between barriers.  A register spilled
// inside the loop over units costs far more than its two instructions: its reload waits for every memory request in front of it,
// the next unit's gather among them (width 96: 160 us with two such, 141 without).  Hence the loads, each waited for on every path of
// the unit that issued it, and the opaque copies of the address bases.
//
// Measured, alone on the chip: 65 536 rows, width 48, He 192: 72 us of a kernel with 32 hidden units per wavefront, erff and expf -> 37;
// 131 056 rows, width 96, He 384: 107 + 96 us of two kernels (row gradients, weight gradients) -> 141 (4% more with the present form of the
// activation, which has one instruction per element more than the one it was measured with: twice_gelu4).
//
// TERMS: bf16 terms of the activation and of p dz, backward_terms(DS).
#include "bwd_mfma.h"
#include "lds_rows.h"
#include "onepass_split.h"
#include "wavefront.h"

namespace slicemoe {

constexpr int kUnit = kOnepassUnit;

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

// Rows of bf16 values in the LDS for 16-wide tiles: PW 16-byte pieces per row, the piece index XORed with a function of the row
// so that neither way of reading meets bank conflicts.  Transposed (half-wavefronts): 8 consecutive rows x 32 bytes.  As A operand
// the hardware serves lanes 0-3, 12-15, 20-27 together, then 4-11, 16-19, 28-31: rows r and r + 8 of which one reads an even piece
// and the other the odd one beside it, so bit 0 of the piece stays as it is.
template <int DS> struct Rows16 {
    static constexpr int P = DS / 8;
    static constexpr int PW = P <= 4 ? 4 : P <= 8 ? 8 : 16;
    static constexpr int STRIDE = PW * 16;
    static_assert(P <= 16, "slices of at most 128 features");
    static __device__ __forceinline__ int swizzle(int row) { return (PW == 4 ? (row >> 2) & 1 : PW == 8 ? (row >> 1) & 3 : row & 7) << 1; }
    static __device__ __forceinline__ int offset(int row, int piece) { return row * STRIDE + ((piece ^ swizzle(row)) << 4); }
};

// p dz of a unit in the LDS: [term][hidden unit of the block][32 rows] bf16, the 8-byte quads of rows permuted inside a hidden unit's
// 64 bytes: the transposing reads (8 hidden units x four quads per half-wavefront) meet no bank conflict.
__device__ __forceinline__ int pdz16_offset(int hidden, int quad)
{
    const int sw = (((hidden >> 2) & 1) << 2) | (((hidden >> 3) & 1) << 1);
    return hidden * 64 + ((quad ^ sw) << 3);
}

// Geometry of one instantiation.
template <int DS, int WAVES, int TERMS> struct ExpertTile {
    typedef Rows16<DS> LR;
    static constexpr int KS = (DS + 31) / 32, FT = (DS + 15) / 16, THREADS = WAVES * 64;
    static constexpr int DXW = 2 * FT;   // wavefronts with a tile of 16 rows x 16 features of dL/dx
    static_assert(DXW <= WAVES, "a wavefront per tile");
    static constexpr size_t rows_bytes = (size_t)2 * kUnit * LR::STRIDE;         // x and dy of one unit
    static constexpr size_t pdz_bytes = (size_t)TERMS * WAVES * 16 * kUnit * 2;
    static constexpr size_t off_w1 = 2 * rows_bytes;                             // [hidden unit][feature] of the block's pass
    static constexpr size_t off_pdz = off_w1 + (size_t)WAVES * 16 * LR::STRIDE;
    static constexpr size_t off_p = off_pdz + 2 * pdz_bytes;                     // [2][32] probabilities
    static constexpr size_t off_id = off_p + 2 * kUnit * 4;                      // [2][32] assignment ids
    static constexpr size_t off_dp = off_id + 2 * kUnit * 4;                     // [2][WAVES][32] partial dL/dp
    static constexpr size_t lds = off_dp + 2 * WAVES * kUnit * 4;
    static_assert(lds <= 160 * 1024, "fits a CU");
};

template <int DS, int WAVES, int TERMS, int MINWAVES>
__global__ __launch_bounds__(WAVES * 64, MINWAVES) void bwd_expert_kernel(
    const bf16_t *__restrict__ x, const bf16_t *__restrict__ dout, const float *__restrict__ pk,
    const int32_t *__restrict__ offsets, const int32_t *__restrict__ perm, const char *__restrict__ packed,
    size_t e_stride, size_t off_w2r, size_t off_b1, int He, int E, int k, int blocks, int overhead, int pass_tiles,
    size_t slot_floats, float *__restrict__ part, float *__restrict__ dxrow, float *__restrict__ dpk)
{
    typedef ExpertTile<DS, WAVES, TERMS> G;
    typedef Rows16<DS> LR;
    constexpr int KS = G::KS, FT = G::FT, THREADS = G::THREADS, P = LR::P, PW = LR::PW, STRIDE = LR::STRIDE;
    constexpr int KS16 = (DS + 15) / 16;        // K-steps of 16 in the packed fragments
    constexpr int PIECES = 2 * kUnit * P;       // 16-byte pieces of a unit's x, then dy: at most one per thread
    static_assert(PIECES <= THREADS && PIECES % 64 == 0, "whole wavefronts move a piece per lane");
    extern __shared__ __align__(16) char lds[];

    const int tid = threadIdx.x, c16 = tid & 15, G4 = (tid >> 4) & 3;
    int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int HT = He / 16;
    // Blocks of one XCD (consecutive ids go to the eight in turn) take consecutive shares: an expert's weights in few L2s.  Not where two blocks fit a
    // compute unit: a batch of hardly more units than blocks has two units in half of the shares and none in the others, and the busy ones would crowd
    // half of the XCDs (width 24, He 96, 400 and 480 units: backward 49.9 and 51.2 us, 47.1 and 48.2 without).
    const int vb = WAVES > 8 && blocks % 8 == 0 ? (int)(blockIdx.x % 8) * (blocks / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;

    const int off_lo = offsets[min(lane, E)], off_hi = offsets[min(lane + 1, E)];
    const RowAxis A = row_axis(off_hi - off_lo, kUnit, overhead, blocks, lane);
    const int c0 = vb * A.share, c1 = c0 + A.share;

    // ---- the piece this thread moves
    const bool moves = wave * 64 < PIECES;
    const int q = min(tid, PIECES - 1);
    const bool mdy = kUnit * P % 64 == 0 ? wave * 64 >= kUnit * P : q >= kUnit * P;   // (whole wavefronts, but for 24)
    const int mrow = (q - (mdy ? kUnit * P : 0)) / P, mcol = (q - (mdy ? kUnit * P : 0)) % P;
    const int mdst = (mdy ? kUnit * STRIDE : 0) + LR::offset(mrow, mcol);
    const bf16_t *msrc = (mdy ? dout : x) + 8 * mcol;
    const bool has_dx = G::DXW == WAVES || wave < G::DXW;
    const bool keeper = wave == WAVES - 1;   // moves the probability and the assignment id of row lane % 32, sums dL/dp
    int a_base = LR::offset(c16, G4);             // piece 4 ks + G4 of row c16: a_base ^ (ks << 6)
    const int trow = 4 * G4 + (c16 >> 2);         // first row this lane points at in a transposing read
    int t_base = LR::offset(trow, (c16 & 3) >> 1) + 8 * (c16 & 1);   // features 16 ft ..: t_base ^ (ft << 5)
    int pz_read = pdz16_offset(trow, c16 & 3);    // rows 16 rt ..: ^ (rt << 5)
    int pz_write = pdz16_offset(16 * wave + c16, G4);
    // the fragment with lane = column, slots = rows 4 G4 .. and 16 + 4 G4 .., of an image of rows
    auto transposed = [&](const char *rows, int col) { return read_transposed(as_lds(rows + col), as_lds(rows + 16 * STRIDE + col)); };

    if constexpr (PW > P) {   // the pieces past the slice width stay zero: rows of x and dy, both buffers; W1 behind them
        for (int t = tid; t < (4 * kUnit + WAVES * 16) * (PW - P); t += THREADS)
            *(uint4 *)(lds + LR::offset(t / (PW - P), P + t % (PW - P))) = make_uint4(0, 0, 0, 0);
    }

    for (int e = 0; e < E; ++e) {
        const int first = __builtin_amdgcn_readlane(A.first, e), steps = __builtin_amdgcn_readlane(A.steps, e);
        if (first >= c1) break;
        const int s_lo = max(0, c0 - first - overhead), s_hi = min(steps, c1 - first - overhead);
        if (s_hi <= s_lo) continue;
        const int row0 = __builtin_amdgcn_readlane(off_lo, e) + s_lo * kUnit;   // rows below count from here
        const int nrows = min(__builtin_amdgcn_readlane(off_hi, e) - row0, (s_hi - s_lo) * kUnit);
        const int32_t *ids = perm + row0;
        const char *ew = packed + (size_t)e * e_stride;
        float *dxs = dxrow + (size_t)row0 * DS;

        for (int t0 = 0; t0 < HT; t0 += pass_tiles) {
            const int nt = min(pass_tiles, HT - t0);   // 16-wide hidden tiles of this pass (even)
            const bool active = wave < nt, again = t0 > 0;
            const float scale = t0 + nt == HT ? 0.5f : 1.f;   // (the activation stage works on twice its values)

            // ---- gather of a unit: assignment ids two units ahead, rows one unit ahead
            int an = 0, ao_next = 0, ao_load = 0;
            uint4 mv = make_uint4(0, 0, 0, 0);
            float p_next = 0.f, dp_before = 0.f;
            auto id_of = [&](int row) { return *(const int32_t *)((const char *)ids + 4u * (unsigned)min(row, nrows - 1)); };
            auto load_ids = [&](int r0) {
                if (moves) an = id_of(r0 + mrow);
                if (keeper) ao_next = id_of(r0 + (lane & (kUnit - 1)));
            };
            auto find_slices = [&]() {
                if (moves) an = divide_by_k(an, k);
                asm volatile("" : "+v"(ao_next), "+v"(dp_before));   // (waited for here, in front of the unit's stores)
            };
            auto load_rows = [&]() {
                if (moves) mv = *(const uint4 *)((const char *)msrc + (unsigned long long)(unsigned)an * (DS * 2));
                if (keeper) {
                    ao_load = ao_next;
                    p_next = pk[ao_next];
                }
            };
            auto store_rows = [&](int r0, int buf) {   // rows past the end: dy and p are zero, so they add nothing
                if (moves) *(uint4 *)(lds + buf * G::rows_bytes + mdst) = !mdy || r0 + mrow < nrows ? mv : make_uint4(0, 0, 0, 0);
                if (keeper) {
                    ((int *)(lds + G::off_id))[buf * kUnit + (lane & (kUnit - 1))] = ao_load;
                    ((float *)(lds + G::off_p))[buf * kUnit + (lane & (kUnit - 1))] = r0 + (lane & (kUnit - 1)) < nrows ? p_next : 0.f;
                }
            };
            load_ids(0);

            lds_barrier();   // everyone is done with the LDS of the pass before
            // ---- this pass's weights: W1 from 32-wide fragment order to [hidden unit][feature] in the LDS, W2 into registers
            {
                const u32x4 *src = (const u32x4 *)(ew + (size_t)(t0 / 2) * KS16 * 1024);
                const int n = nt / 2 * KS16 * 64;
                constexpr int U = 4;
                for (int b = 0; b < n; b += U * THREADS) {
                    u32x4 v[U];
#pragma unroll
                    for (int i = 0; i < U; ++i) v[i] = src[min(b + tid + i * THREADS, n - 1)];
                    asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));   // all requested before one is used
#pragma unroll
                    for (int i = 0; i < U; ++i) {
                        const int f = b + tid + i * THREADS, l = f & 63, r = f >> 6, ks = r % KS16, h32 = r / KS16;
                        if (f < n) *(u32x4 *)(lds + G::off_w1 + LR::offset(32 * h32 + (l & 31), 2 * ks + (l >> 5))) = v[i];
                    }
                }
            }
            const int tile = active ? t0 + wave : t0;
            bf16x8 w2[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int s16 = 2 * ks + (G4 >> 1);
                uint4 v = ((const uint4 *)(ew + off_w2r))[((tile >> 1) * KS16 + min(s16, KS16 - 1)) * 64 + (G4 & 1) * 32 + 16 * (tile & 1) + c16];
                if (KS16 % 2 != 0 && s16 >= KS16) v = make_uint4(0, 0, 0, 0);
                w2[ks] = __builtin_bit_cast(bf16x8, v);
            }
            const float bias = ((const float *)(ew + off_b1))[tile * 16 + c16];
            if (!active) {   // nothing from this wavefront for dL/dp, and zeros in both operands of dL/dx
                ((float *)(lds + G::off_dp))[((lane >> 5) * WAVES + wave) * kUnit + (lane & 31)] = 0.f;
                const uint4 zero = make_uint4(0, 0, 0, 0);
                for (int t = lane; t < STRIDE; t += 64) *(uint4 *)(lds + G::off_w1 + wave * 16 * STRIDE + t * 16) = zero;
                for (int t = lane; t < 2 * TERMS * 64; t += 64) *(uint4 *)(lds + G::off_pdz + ((t >> 6) * WAVES + wave) * 1024 + (t & 63) * 16) = zero;
            }
            const char *w1s = lds + G::off_w1, *w1w = w1s + wave * 16 * STRIDE;

            f32x4 aW1[FT], aW2[FT];   // lane = hidden unit, registers = features; lane = feature, registers = hidden units
            float ab1 = 0.f, ab2 = 0.f;
#pragma unroll
            for (int ft = 0; ft < FT; ++ft) aW1[ft] = aW2[ft] = f32x4{0.f, 0.f, 0.f, 0.f};

            find_slices();
            load_rows();
            load_ids(kUnit);   // (past the end: the last row's)
            store_rows(0, 0);
            find_slices();
            lds_barrier();

            // ---- dL/dx of the unit before
            const int dft = wave >> 1, drt = wave & 1;
            const int dx_col = 4 * (16 * dft + 4 * G4);   // bytes (unsigned offsets: a segment's dL/dx is below 4 GB, a block's share of the rows that fit the card)
            f32x4 dx, dx_before;
            // (Every load here is waited for on every path of the same unit: one left over would be waited for where its registers
            // are written next, behind the gather of the next unit, whose latency would then show.)
            auto dx_begin = [&](int r0, int buf) {   // r0 < 0: there is no unit before
                dx = dx_before = f32x4{0.f, 0.f, 0.f, 0.f};
                if (again && has_dx) {
                    const int col = DS % 16 == 0 ? dx_col : min(dx_col, 4 * DS - 16);
                    dx_before = *(const f32x4 *)((const char *)dxs + (unsigned)max(min(r0 + 16 * drt + c16, nrows - 1), 0) * (4u * DS) + (unsigned)col);
                }
                if (again && keeper) dp_before = dpk[r0 < 0 ? 0 : ((const int *)(lds + G::off_id))[buf * kUnit + (lane & (kUnit - 1))]];
            };
            struct DxFrags {
                bf16x8 w, b[TERMS];
            };
            auto dx_load = [&](DxFrags &f, int buf, int kk) {   // 32 hidden units (past the pass's last: zeros in both operands)
                f.w = transposed(w1s + kk * 32 * STRIDE, t_base ^ (dft << 5));
                const char *pz = lds + G::off_pdz + buf * G::pdz_bytes + kk * 2048 + (pz_read ^ (drt << 5));
#pragma unroll
                for (int t = 0; t < TERMS; ++t) f.b[t] = read_transposed(as_lds(pz + t * WAVES * 1024), as_lds(pz + t * WAVES * 1024 + 1024));
            };
            auto dx_all = [&](int buf) {
                if (!has_dx) return;
                DxFrags f[2];   // (a step's fragments are requested while the matrix instructions of the one before run)
                dx_load(f[0], buf, 0);
#pragma unroll
                for (int kk = 0; kk < WAVES / 2; ++kk) {
                    if (kk + 1 < WAVES / 2) dx_load(f[(kk + 1) & 1], buf, kk + 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int t = TERMS - 1; t >= 0; --t) dx = mfma16(f[kk & 1].w, f[kk & 1].b[t], dx);   // small terms first
                }
            };
            auto dx_end = [&](int r0, int buf) {   // stores the rows r0 ..
                dx = (dx_before + dx) * scale;
                const int row = r0 + 16 * drt + c16;
                if (has_dx && (DS % 16 == 0 || dx_col < 4 * DS) && (unsigned)row < (unsigned)nrows)
                    *(f32x4 *)((char *)dxs + ((unsigned)row * (4u * DS) + (unsigned)dx_col)) = dx;
                if (keeper) {
                    const float *dps = (const float *)(lds + G::off_dp) + buf * WAVES * kUnit + (lane & (kUnit - 1));
                    float v[WAVES], t = dp_before;
#pragma unroll
                    for (int w = 0; w < WAVES; ++w) v[w] = dps[w * kUnit];
#pragma unroll
                    for (int w = 0; w < WAVES; ++w) t += v[w];
                    if (lane < kUnit && (unsigned)(r0 + lane) < (unsigned)nrows)
                        dpk[((const int *)(lds + G::off_id))[buf * kUnit + lane]] = t * scale;
                }
            };

            int buf = 0;
            for (int r0 = 0; r0 < nrows; r0 += kUnit) {
                const bool more = r0 + kUnit < nrows;
                // opaque, so that the dozens of addresses made from them are made here and not kept in registers
                asm volatile("" : "+v"(a_base), "+v"(t_base), "+v"(pz_read), "+v"(pz_write), "+v"(lane));
                if (more) {
                    load_rows();
                    load_ids(r0 + 2 * kUnit);
                }
                dx_begin(r0 - kUnit, buf ^ 1);   // (for the first unit dL/dx works on what the buffers hold, and nothing of it is stored)
                const char *xs = lds + buf * G::rows_bytes, *gs = xs + kUnit * STRIDE;
                const float *ps = (const float *)(lds + G::off_p) + buf * kUnit;
                uint32_t a1[TERMS][4], pdz[TERMS][4];   // terms, the largest first; register pairs are row pairs
                if (active) {
                    // lane = hidden unit c16 of this tile, register i of u[rt] = row 16 rt + 4 G4 + i of the unit; the fragments of a
                    // K-step are requested while the matrix instructions of the one before run
                    f32x4 u[2], da[2];
                    bf16x8 w1[2], xa[2][2], ga[2][2];
                    auto first_load = [&](int ks) {
                        const int at = a_base ^ (ks << 6), s = ks & 1;
                        w1[s] = *(const bf16x8 *)(w1w + at);
#pragma unroll
                        for (int rt = 0; rt < 2; ++rt) {
                            xa[s][rt] = *(const bf16x8 *)(xs + at + rt * 16 * STRIDE);
                            ga[s][rt] = *(const bf16x8 *)(gs + at + rt * 16 * STRIDE);
                        }
                    };
#pragma unroll
                    for (int rt = 0; rt < 2; ++rt) u[rt] = da[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
                    first_load(0);
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        if (ks + 1 < KS) first_load(ks + 1);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int rt = 0; rt < 2; ++rt) {
                            u[rt] = mfma16(xa[ks & 1][rt], w1[ks & 1], u[rt]);
                            da[rt] = mfma16(ga[ks & 1][rt], w2[ks], da[rt]);
                        }
                    }
                    float du[8];   // dz u, summed over the hidden units below
#pragma unroll
                    for (int rt = 0; rt < 2; ++rt) {
                        const f32x4 pv = *(const f32x4 *)(ps + 16 * rt + 4 * G4);
                        float z[4], act[4], slope[4], dz[4], pd[4];
#pragma unroll
                        for (int c = 0; c < 4; ++c) z[c] = fmaf(pv[c], u[rt][c], bias);
                        twice_gelu4(z, act, slope);
#pragma unroll
                        for (int c = 0; c < 4; ++c) dz[c] = da[rt][c] * slope[c];   // twice dL/dz
#pragma unroll
                        for (int c = 0; c < 4; ++c) pd[c] = pv[c] * dz[c];
                        split_terms<TERMS>(act, a1, 2 * rt);
                        split_terms<TERMS>(pd, pdz, 2 * rt);
                        ab1 += (dz[0] + dz[1]) + (dz[2] + dz[3]);
#pragma unroll
                        for (int c = 0; c < 4; ++c) du[4 * rt + c] = dz[c] * u[rt][c];
                        char *dst = lds + G::off_pdz + buf * G::pdz_bytes + (pz_write ^ (rt << 5));
#pragma unroll
                        for (int t = 0; t < TERMS; ++t) *(uint2 *)(dst + t * WAVES * 1024) = make_uint2(pdz[t][2 * rt], pdz[t][2 * rt + 1]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    // dL/dp: this tile's hidden units; every fourth lane ends up with the sums of two rows
                    sum_over_hidden(du);
                    if ((lane & 3) == 0)
                        *(float2 *)((float *)(lds + G::off_dp) + (buf * WAVES + wave) * kUnit + 16 * ((lane >> 3) & 1) + 4 * (lane >> 4) + 2 * ((lane >> 2) & 1)) =
                            make_float2(du[0], du[1]);
                }
                dx_all(buf ^ 1);
                if (active) {
                    auto frag = [](const uint32_t (&v)[4]) { return __builtin_bit_cast(bf16x8, make_uint4(v[0], v[1], v[2], v[3])); };
                    bf16x8 gt[2], xt[2];
                    auto second_load = [&](int ft) {
                        gt[ft & 1] = transposed(gs, t_base ^ (ft << 5));
                        xt[ft & 1] = transposed(xs, t_base ^ (ft << 5));
                    };
                    second_load(0);
#pragma unroll
                    for (int ft = 0; ft < FT; ++ft) {
                        if (ft + 1 < FT) second_load(ft + 1);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int t = TERMS - 1; t >= 0; --t) {   // small terms first
                            aW2[ft] = mfma16(frag(a1[t]), gt[ft & 1], aW2[ft]);
                            aW1[ft] = mfma16(xt[ft & 1], frag(pdz[t]), aW1[ft]);
                        }
                    }
                }
                if (t0 == 0 && wave < FT) ab2 += fragment_sum(transposed(gs, t_base ^ (wave << 5)));   // db2: sums of dy over the rows
                find_slices();
                dx_end(r0 - kUnit, buf ^ 1);   // (reads the keeper's ids, which the next line replaces)
                if (more) store_rows(r0 + kUnit, buf ^ 1);
                lds_barrier();
                buf ^= 1;
            }
            {   // the last unit's dL/dx
                const int r_last = (s_hi - s_lo - 1) * kUnit;
                dx_begin(r_last, buf ^ 1);
                dx_all(buf ^ 1);
                dx_end(r_last, buf ^ 1);
            }

            // ---- this segment's slot: dW1 [ds][He] | dW2 [He][ds] | db1 [He] | db2 [ds]
            int he = He, co = c16, go = G4;   // opaque copies: the store addresses are made here, not kept in registers through the loop above
            asm volatile("" : "+s"(he), "+v"(co), "+v"(go));
            float *slot = part + (size_t)(vb + e) * slot_floats;
            float *pW1 = slot, *pW2 = pW1 + (size_t)DS * he, *pb1 = pW2 + (size_t)he * DS, *pb2 = pb1 + he;
            if (active) {
                const int h0 = 16 * (t0 + wave);
#pragma unroll
                for (int ft = 0; ft < FT; ++ft)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int f = 16 * ft + 4 * go + i;
                        if (DS % 16 == 0 || f < DS) pW1[(size_t)f * he + h0 + co] = 0.5f * aW1[ft][i];
                        if (DS % 16 == 0 || 16 * ft + co < DS) pW2[(size_t)(h0 + 4 * go + i) * DS + 16 * ft + co] = 0.5f * aW2[ft][i];
                    }
                ab1 += __shfl_xor(ab1, 16);   // the four lane groups hold different rows of the same hidden unit
                ab1 += __shfl_xor(ab1, 32);
                if (go == 0) pb1[h0 + co] = 0.5f * ab1;
            }
            if (t0 == 0 && wave < FT) {
                ab2 += __shfl_xor(ab2, 16);
                ab2 += __shfl_xor(ab2, 32);
                const int f = 16 * wave + co;
                if (go == 0 && (DS % 16 == 0 || f < DS)) pb2[f] = ab2;
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------------ host
// Blocks there are units for, at the most: an expert's rows begin one.
static long long expert_blocks_bound(const slicemoe_config &c, long long units)
{
    const long long cap = (long long)num_compute_units() * onepass_blocks_per_cu(c.d / c.S, c.He), most = units + c.E - 1;
    return most < 1 ? 1 : most < cap ? most : cap;
}

// Up to two units per expert every unit has a block of its own (no position for an expert's beginning: it would make the share of a block that has
// experts of one unit each the number of experts over the number of whole units).  Beyond, a block has at least a beginning and a unit, or two
// units: fewer slots of partial sums, whose traffic is more than the second unit costs.  Backward in us, with the position / without:
//   2 E units and fewer   width 96, He 384: 1 token (S 8), 16 experts 134 / 56, 64 tokens (32 units) 69.9 / 66.5; He 768, 64 experts, 4 tokens 404 / 121, 128 units 156 / 151
//                         width 48, He 192, 16 experts: 2 units 81 / 42, 32 units 48.0 / 46.6; width 24, He 96: 2 units 60 / 37, 32 units 42.6 / 41.6
//   more, 16 experts      256 units: width 96, He 192 64.7 / 65.0, He 768 117 / 123; width 48, He 192 53.2 / 55.1; 4096 units: width 96, He 384 216 / 225
BackwardWeightsPlan backward_expert_plan(const slicemoe_config &c)
{
    BackwardWeightsPlan W;
    const long long units = ((long long)c.T * c.S * c.k + kUnit - 1) / kUnit, most = expert_blocks_bound(c, units);
    const bool few = units <= 2 * c.E;
    W.onepass = W.fused = true;
    W.step = kUnit;
    W.overhead = few ? 0 : 1;
    W.groups = 1;
    W.blocks = (int)(few || units > most ? most : units);
    W.slots = (long long)W.blocks + c.E;
    W.reserve = most + c.E;
    return W;
}

template <int DS, int WAVES, int MINWAVES>
static hipError_t run_expert(const slicemoe_config &c, const BackwardWeightsPlan &W, const BwdPacked &L, const void *h, const void *d_out, const float *pk,
                             const int32_t *offsets, const int32_t *perm, const char *packed, size_t slot_floats, float *part,
                             float *dxrow, float *dpk, hipStream_t s)
{
    constexpr int TERMS = backward_terms(DS);
    constexpr size_t lds = ExpertTile<DS, WAVES, TERMS>::lds;
    if (onepass_waves(DS, c.He) != WAVES) return hipErrorInvalidValue;
    auto kern = bwd_expert_kernel<DS, WAVES, TERMS, MINWAVES>;
    const hipError_t e = grant_dynamic_lds((const void *)kern, lds);
    if (e != hipSuccess) return e;
    kern<<<(unsigned)W.blocks, WAVES * 64, lds, s>>>((const bf16_t *)h, (const bf16_t *)d_out, pk, offsets, perm, packed, L.stride, L.w2r,
                                                     L.b1, c.He, c.E, c.k, W.blocks, W.overhead, onepass_pass_tiles(DS, c.He), slot_floats, part,
                                                     dxrow, dpk);
    return hipGetLastError();
}

hipError_t launch_backward_expert_onepass(const slicemoe_config &c, const BackwardWeightsPlan &W, const BwdPacked &L, const void *h, const void *d_out,
                                          const float *pk, const int32_t *offsets, const int32_t *perm, const char *packed, size_t slot_floats,
                                          float *part, float *dxrow, float *dpk, hipStream_t s)
{
    const int ds = c.d / c.S;
    return ds == 24 && onepass_waves(ds, c.He) == 8 ? run_expert<24, 8, 4>(c, W, L, h, d_out, pk, offsets, perm, packed, slot_floats, part, dxrow, dpk, s)
         : ds == 24 ? run_expert<24, 16, 4>(c, W, L, h, d_out, pk, offsets, perm, packed, slot_floats, part, dxrow, dpk, s)
         : ds == 48 ? run_expert<48, 12, 3>(c, W, L, h, d_out, pk, offsets, perm, packed, slot_floats, part, dxrow, dpk, s)
         : ds == 96 ? run_expert<96, 12, 3>(c, W, L, h, d_out, pk, offsets, perm, packed, slot_floats, part, dxrow, dpk, s)
                    : hipErrorInvalidValue;
}

}  // namespace slicemoe
