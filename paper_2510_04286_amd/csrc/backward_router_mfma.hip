// Matrix-core backward of the router and assembly of dL/dh, for the forward's matrix-core slice widths except 384,
// Hr = 256 and up to 64 experts.  Same mathematics as bwd_router_generic_kernel in backward_generic.hip; three kernels, the first two in one
// (bwd_route_slices_mfma_kernel) where the LDS holds the fragments of both: widths 24, 48 and 64, and 96 with up to 32 experts:
//
//   bwd_route_logits_mfma_kernel   the forward router's layout: a lane owns one slice of a 32-slice tile.  Recomputes the
//       router: the hidden layer exactly as the forward does (bf16 MFMA with the bias preloaded: the same ReLU pattern), the
//       logits to fp32 rounding (ReLU and two-term fp16 split on fp16 MFMA like the forward's, or three bf16 terms on bf16
//       MFMA, see below); noise; softmax with the temperature; then per lane: the selected probabilities, back
//       through the dropout's renormalisation and the softmax to dL/dg (16 experts per lane and expert tile, as the
//       logits).  Writes dL/dg as bf16 tables, one per term, and the ReLU pattern, one bit per hidden unit.
//   bwd_route_inputs_mfma_kernel   same layout: dL/du = Wr2 dL/dg with dL/dg read back in accumulator order, i.e. as
//       the B operand, masked by the ReLU bits, then dL/dx += Wr1 dL/du chained from registers.  Writes
//       dL/dh = that + the k expert-path rows of the slice (one bf16 rounding).
//   bwd_route_weights_mfma_kernel  the transposed layout (see backward_weights_mfma.hip): one wavefront per hidden tile walks
//       the slices of its block.  Stores its pieces into the block's slot of partial sums.
//
// dL/dg, u and dL/du enter matrix instructions as two bf16 terms (16 significant bits) at widths 64, 96 and 128, as three (24
// bits: the fp32 values themselves) at 24, 48 and 192 (kRbTerms).  At the latter the logits too are formed from all of u and from
// Wr2 as it is stored, the softmax uses expf, and dWr2 takes the products of all terms: the gradients are as close to 64-bit
// arithmetic as those of the fp32 kernels (relative errors at width 48, 16 384 slices: 1.5e-7 to 2.8e-7).
#include "bwd_mfma.h"
#include "lds_rows.h"

namespace slicemoe {

typedef _Float16 r_h2 __attribute__((ext_vector_type(2)));
typedef _Float16 r_f16x8 __attribute__((ext_vector_type(8)));

constexpr int kRbHr = 256, kRbHT = 8;
constexpr int kRbThreads = 512;                 // slice kernels: 8 wavefronts
constexpr int kRbWaves = kRbThreads / 64;
template <int DS> constexpr int kRbTerms = backward_terms(DS);   // bf16 terms of dL/dg, u and dL/du

// Repacked router (bytes from the start of the buffer); KS = ds / 16 and OT = ds / 32 rounded up (zero-padded), ET = expert tiles of 32 (experts
// past E are zero).
//   w1f  [8][KS][64]      Wr1 fragments, lane (i, g), slot m: Wr1[16ks + 8g + m][32ht + i]                   (bf16)
//   w2f  [8][2][ET][64]   Wr2 for the logits: lane (i, g), slot m: Wr2[32ht + chain(s, g, m)][32et + i]       (fp16; bf16 with three terms)
//   w2c  [ET][2][8][64]   Wr2 for dL/du:      lane (i, g), slot m: Wr2[32ht + i][32et + chain(s, g, m)]       (bf16)
//   w1c  [8][2][OT][64]   Wr1 for dL/dx:      lane (i, g), slot m: Wr1[32ot + i][32ht + chain(s, g, m)]       (bf16)
//   w2r  [8][2 ET][64]    rows of Wr2:        lane (i, g), slot m: Wr2[32ht + i][16s + 8g + m]                (bf16)
//   b1 [256] fp32, b2 [32 ET] fp32
struct RouterBwdPacked {
    size_t w1f, w2f, w2c, w1c, w2r, b1, b2, total;
};
static RouterBwdPacked router_bwd_layout(int ds, int ET)
{
    RouterBwdPacked L;
    const int KS = (ds + 15) / 16, OT = (ds + 31) / 32;
    size_t at = 0;
    L.w1f = at;  at += (size_t)kRbHT * KS * 1024;
    L.w2f = at;  at += (size_t)ET * kRbHT * 2 * 1024;
    L.w2c = at;  at += (size_t)ET * 2 * kRbHT * 1024;
    L.w1c = at;  at += (size_t)kRbHT * 2 * OT * 1024;
    L.w2r = at;  at += (size_t)kRbHT * 2 * ET * 1024;
    L.b1 = at;   at += (size_t)kRbHr * 4;
    L.b2 = at;   at += 256;
    L.total = at;
    return L;
}

// ------------------------------------------------------------------------------------------ stages of the slice kernels
// ReLU of a hidden pre-activation, at most twice the largest fp16 value (what the two fp16 terms of the hidden layer can hold): a median
// takes its operands as they are, where a maximum would first spend an instruction on quieting one.  0 for NaN; +Inf is capped too, see
// split_pair_f16.
__device__ __forceinline__ float relu_capped(float a) { return __builtin_amdgcn_fmed3f(a, 0.f, 131008.f); }
// The ReLU pattern of 32 hidden units in one word, the first unit in the top bit: shifted up by one with the bit of a unit below
// (r >= 0 is above zero exactly if adding 2^31 - 1 to its bit pattern reaches the sign bit).
__device__ __forceinline__ uint32_t push_active(uint32_t bits, float r)
{
    return __builtin_amdgcn_alignbit(bits, (uint32_t)__float_as_int(r) + 0x7fffffffu, 31);
}
// Two-term fp16 split of the ReLU of a pair of pre-activations a0, a1, whose capped ReLU is r0, r1: the round-toward-zero conversion of the
// pair, negative halves (and NaN) to zero, and per activation one mixed-precision multiply-add r - u0 rounded to fp16.  An infinite
// pre-activation stays one in the first term, as in the forward's router, and its second is -Inf: NaN in the logits of the slice, and so in its
// gradients.  (The first term from r0, r1 would be 65504: finite gradients of a slice whose output is not.)
__device__ __forceinline__ void split_pair_f16(float a0, float a1, float r0, float r1, uint32_t &u0, uint32_t &u1)
{
    const r_h2 hi = __builtin_elementwise_max(__builtin_bit_cast(r_h2, __builtin_amdgcn_cvt_pkrtz(a0, a1)), r_h2{0, 0});
    u0 = __builtin_bit_cast(uint32_t, hi);
    asm("v_fma_mixlo_f16 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(u1) : "v"(u0), "v"(r0));
    asm("v_fma_mixhi_f16 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(u1) : "v"(u0), "v"(r1));
}

// The forward router for one slice per lane pair: logits in accumulator order, and which hidden units are active (word w: hidden tiles
// 2w and 2w + 1, accumulator order).  w1f [8][KS][64], w2f [8][2][ET][64], b1s [256], b2s [32 ET].
template <int DS, int ET>
__device__ __forceinline__ void router_logits(const bf16x8 (&xb)[SliceTiles<DS>::KS], const uint4 *w1f, const uint4 *w2f, const float *b1s,
                                              const float *b2s, int lane, int g, f32x16 (&gacc)[ET], uint32_t (&act)[4])
{
    constexpr int KS = SliceTiles<DS>::KS, TERMS = kRbTerms<DS>;
#pragma unroll
    for (int et = 0; et < ET; ++et)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 b = *(const f32x4 *)(b2s + et * 32 + 8 * q + 4 * g);
#pragma unroll
            for (int c = 0; c < 4; ++c) gacc[et][4 * q + c] = b[c];
        }
    act[0] = act[1] = act[2] = act[3] = 0;
#pragma unroll 1
    for (int hp = 0; hp < kRbHT; hp += 2) {
        uint32_t bits = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ht = hp + h;
            f32x16 acc;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 b = *(const f32x4 *)(b1s + ht * 32 + 8 * q + 4 * g);
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[4 * q + c] = b[c];
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) acc = mfma_bf16(__builtin_bit_cast(bf16x8, w1f[(ht * KS + ks) * 64 + lane]), xb[ks], acc);
            if constexpr (TERMS == 3) {   // the hidden layer whole, against the bf16 weights as they are
                uint32_t ut[2][TERMS][4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float u[4] = {fmaxf(acc[4 * q], 0.f), fmaxf(acc[4 * q + 1], 0.f), fmaxf(acc[4 * q + 2], 0.f), fmaxf(acc[4 * q + 3], 0.f)};
#pragma unroll
                    for (int c = 0; c < 4; ++c) bits = push_active(bits, u[c]);
                    split_terms<TERMS>(u, ut[q >> 1], 2 * (q & 1));
                }
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int et = 0; et < ET; ++et) {
                        const bf16x8 a2 = __builtin_bit_cast(bf16x8, w2f[((ht * 2 + s) * ET + et) * 64 + lane]);
#pragma unroll
                        for (int t = TERMS - 1; t >= 0; --t)   // small terms first
                            gacc[et] = mfma_bf16(a2, __builtin_bit_cast(bf16x8, make_uint4(ut[s][t][0], ut[s][t][1], ut[s][t][2], ut[s][t][3])), gacc[et]);
                    }
            } else {
                uint32_t t0[8], t1[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float r0 = relu_capped(acc[2 * i]), r1 = relu_capped(acc[2 * i + 1]);
                    bits = push_active(push_active(bits, r0), r1);
                    split_pair_f16(acc[2 * i], acc[2 * i + 1], r0, r1, t0[i], t1[i]);
                }
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const r_f16x8 u0 = __builtin_bit_cast(r_f16x8, make_uint4(t0[4 * s], t0[4 * s + 1], t0[4 * s + 2], t0[4 * s + 3]));
                    const r_f16x8 u1 = __builtin_bit_cast(r_f16x8, make_uint4(t1[4 * s], t1[4 * s + 1], t1[4 * s + 2], t1[4 * s + 3]));
#pragma unroll
                    for (int et = 0; et < ET; ++et) {
                        const r_f16x8 a2 = __builtin_bit_cast(r_f16x8, w2f[((ht * 2 + s) * ET + et) * 64 + lane]);
                        gacc[et] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a2, u1, gacc[et], 0, 0, 0);   // small term first
                        gacc[et] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a2, u0, gacc[et], 0, 0, 0);
                    }
                }
            }
        }
        act[0] = act[1];   // (the words move up: after four pairs the first is in front)
        act[1] = act[2];
        act[2] = act[3];
        act[3] = bits;
    }
}

// What a slice's gradient needs from memory beside its row (both lanes of a slice hold the same selections), requested ahead: of its first
// two assignments (further ones are fetched where they are used).
constexpr int kRbAhead = 2;
template <int ET> struct SliceDraws {
    float noise[ET * 16];                 // of this lane's experts
    int e[kRbAhead], row[kRbAhead];       // the selected experts, their stacked rows (negative: dropped by the capacity limit)
    float dp[kRbAhead], u[kRbAhead];      // dL/dp, the dropout's draws
};
template <int ET>
__device__ __forceinline__ void load_draws(SliceDraws<ET> &D, long long n, int g, int E, int k, const float *__restrict__ noise,
                                           const float *__restrict__ drop_u, const int32_t *__restrict__ idx, const int32_t *__restrict__ inv,
                                           const float *__restrict__ dpk)
{
    asm volatile("" : "+v"(g));   // the addresses are formed here, not kept in registers from tile to tile
    if (noise != nullptr) {
        const float *nr = noise + n * E;
        if ((E & 3) == 0) {   // rows of the table are 16-byte aligned: this lane's four consecutive experts at once
#pragma unroll
            for (int q = 0; q < ET * 4; ++q) {
                const int e0 = (q >> 2) * 32 + 8 * (q & 3) + 4 * g;
                const f32x4 z = *(const f32x4 *)(nr + (e0 < E ? e0 : 0));
#pragma unroll
                for (int c = 0; c < 4; ++c) D.noise[4 * q + c] = z[c];
            }
        } else {
#pragma unroll
            for (int i = 0; i < ET * 16; ++i) D.noise[i] = nr[min((i >> 4) * 32 + acc_feature(i & 15, g), E - 1)];
        }
    }
#pragma unroll
    for (int jj = 0; jj < kRbAhead; ++jj)
        if (jj < k) {
            const long long a = n * k + jj;
            D.e[jj] = idx[a];
            D.row[jj] = inv[a];
            D.dp[jj] = dpk[a];
            if (drop_u != nullptr) D.u[jj] = drop_u[a];
        }
}

// dL/dg of one slice per lane pair from its logits gacc: noise; softmax with the temperature; the selected probabilities, back through
// the dropout's renormalisation and the softmax.  As bf16 pairs in accumulator order, by term.
template <int ET, int TERMS>
__device__ __forceinline__ void logit_gradients(const f32x16 (&gacc)[ET], const SliceDraws<ET> &D, long long n, int g, int E, int k, bool noisy,
                                                float sigma, float inv_tau, const float *__restrict__ drop_u, float rate,
                                                const int32_t *__restrict__ idx, const int32_t *__restrict__ inv, const float *__restrict__ dpk,
                                                bool capped, const float *capg /* [64], LDS */, uint32_t (&dgt)[ET][TERMS][8])
{
    // ---- this lane's 16 ET logits: expert 32 et + acc_feature(r, g); noise; softmax of g / tau over the E experts
    float v[ET * 16];
#pragma unroll
    for (int i = 0; i < ET * 16; ++i) {
        const int e = (i >> 4) * 32 + acc_feature(i & 15, g);
        float t = gacc[i >> 4][i & 15];
        if (noisy) t = fmaf(sigma, D.noise[i], t);
        v[i] = e < E ? t : -INFINITY;
    }
    float m = v[0];
#pragma unroll
    for (int i = 1; i < ET * 16; ++i) m = fmaxf(m, v[i]);
    m = fmaxf(m, __shfl_xor(m, 32));
    const float sc = 1.4426950408889634f * inv_tau, nm = -m * sc;
    float den = 0.f;
#pragma unroll
    for (int i = 0; i < ET * 16; ++i) {
        v[i] = TERMS == 3 ? expf((v[i] - m) * inv_tau) : __builtin_amdgcn_exp2f(fmaf(v[i], sc, nm));
        den += v[i];
    }
    den += __shfl_xor(den, 32);
    const float rden = 1.f / den;
#pragma unroll
    for (int i = 0; i < ET * 16; ++i) v[i] *= rden;   // probability of every expert of this lane's half

    // ---- the k selections: probability, upstream gradient, dropout flag (both lanes of a slice do the same)
    float psel[8], dpf[8];
    bool keep[8];
    int ej[8];
    int kept = 0;
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) {
        psel[jj] = dpf[jj] = 0.f;
        keep[jj] = false;
        ej[jj] = -1;
        if (jj < k) {
            constexpr int LAST = kRbAhead - 1;
            int e = D.e[min(jj, LAST)], row = D.row[min(jj, LAST)];
            float dp = D.dp[min(jj, LAST)], u = D.u[min(jj, LAST)];
            if (jj > LAST) {
                const long long a = n * k + jj;
                e = idx[a];
                row = inv[a];
                dp = dpk[a];
                if (drop_u != nullptr) u = drop_u[a];
                asm volatile("" : "+v"(e), "+v"(row), "+v"(dp), "+v"(u));   // (waited for in this branch, see arrived)
            }
            ej[jj] = e;
            float mine = 0.f;
#pragma unroll
            for (int i = 0; i < ET * 16; ++i) mine = (i >> 4) * 32 + acc_feature(i & 15, g) == ej[jj] ? v[i] : mine;
            psel[jj] = mine + __shfl_xor(mine, 32);     // the expert sits in one of the two halves
            dpf[jj] = row >= 0 ? dp : 0.f;              // a capacity-dropped assignment carries no gradient from h'
            if (capped) dpf[jj] += capg[min(max(ej[jj], 0), E - 1)];   // but it counts as assigned (capacity loss)
            keep[jj] = drop_u != nullptr ? !(u < rate) : true;
            kept += keep[jj] ? 1 : 0;
        }
    }
    if (drop_u != nullptr) {
        if (kept == 0) keep[0] = true;
        float ssum = 0.f, dot = 0.f;
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) ssum += keep[jj] ? psel[jj] : 0.f;
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) dot += keep[jj] ? dpf[jj] * (psel[jj] / ssum) : 0.f;
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) dpf[jj] = keep[jj] ? (dpf[jj] - dot) / ssum : 0.f;
    }
    // dL/dg_e = (1/tau) (sum_j c_j [e = e_j] - p_e sum_j c_j),  c_j = dL/dp_j p_j
    float csum = 0.f;
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) {
        dpf[jj] = jj < k ? dpf[jj] * psel[jj] : 0.f;
        csum += dpf[jj];
    }
#pragma unroll
    for (int i = 0; i < ET * 16; ++i) v[i] = -v[i] * csum;
#pragma unroll
    for (int jj = 0; jj < 8; ++jj)
        if (jj < k) {
#pragma unroll
            for (int i = 0; i < ET * 16; ++i) v[i] += (i >> 4) * 32 + acc_feature(i & 15, g) == ej[jj] ? dpf[jj] : 0.f;
        }
#pragma unroll
    for (int et = 0; et < ET; ++et)
#pragma unroll
        for (int q = 0; q < 4; ++q) {   // experts 32 et + 8q + 4g .. + 3 of this slice: four bf16 values per term
            float dg[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) dg[c] = v[et * 16 + 4 * q + c] * inv_tau;
            uint32_t dt[TERMS][4];
            split_terms<TERMS>(dg, dt, 0);
#pragma unroll
            for (int t = 0; t < TERMS; ++t) {
                dgt[et][t][2 * q] = dt[t][0];
                dgt[et][t][2 * q + 1] = dt[t][1];
            }
        }
}

// dL/dg of a slice in its rows of the tables.
template <int ET, int TERMS>
__device__ __forceinline__ void store_logit_gradients(const uint32_t (&dgt)[ET][TERMS][8], bf16_t *__restrict__ dg_terms, long long Ns, long long n, int g)
{
    constexpr int EP = ET * 32;
#pragma unroll
    for (int et = 0; et < ET; ++et)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int t = 0; t < TERMS; ++t)
                *(uint2 *)(dg_terms + (t * Ns + n) * EP + et * 32 + 8 * q + 4 * g) = make_uint2(dgt[et][t][2 * q], dgt[et][t][2 * q + 1]);
}

// dL/du = Wr2 dL/dg (ReLU pattern applied), dL/dx += Wr1 dL/du, both from registers.  w2c [ET][2][8][64], w1c [8][2][OT][64].
template <int DS, int ET>
__device__ __forceinline__ void input_gradients(const uint32_t (&dgt)[ET][kRbTerms<DS>][8], const uint32_t (&act)[4], const uint4 *w2c, const uint4 *w1c,
                                                int lane, f32x16 (&dx)[SliceTiles<DS>::OT])
{
    constexpr int OT = SliceTiles<DS>::OT, TERMS = kRbTerms<DS>;
#pragma unroll
    for (int ot = 0; ot < OT; ++ot)
#pragma unroll
        for (int i = 0; i < 16; ++i) dx[ot][i] = 0.f;
    uint32_t a0 = act[0], a1 = act[1], a2 = act[2], a3 = act[3];
#pragma unroll 1
    for (int hp = 0; hp < kRbHT; hp += 2) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ht = hp + h;
            f32x16 du;
#pragma unroll
            for (int i = 0; i < 16; ++i) du[i] = 0.f;
#pragma unroll
            for (int et = 0; et < ET; ++et)
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const bf16x8 wf = __builtin_bit_cast(bf16x8, w2c[((et * 2 + s) * kRbHT + ht) * 64 + lane]);
#pragma unroll
                    for (int t = 0; t < TERMS; ++t) du = mfma_bf16(wf, frag_of(dgt[et][t], s), du);   // large terms first, see the weights kernel
                }
            uint32_t dut[2][TERMS][4];   // by K-step
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float d[4];
#pragma unroll
                for (int c = 0; c < 4; ++c)   // the unit's bit, spread over the word, as a mask
                    d[c] = __int_as_float(__float_as_int(du[4 * q + c]) & __builtin_amdgcn_sbfe((int)a0, 31 - 16 * h - 4 * q - c, 1));
                split_terms<TERMS>(d, dut[q >> 1], 2 * (q & 1));
            }
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int ot = 0; ot < OT; ++ot) {
                    const bf16x8 wf = __builtin_bit_cast(bf16x8, w1c[((ht * 2 + s) * OT + ot) * 64 + lane]);
#pragma unroll
                    for (int t = TERMS - 1; t >= 0; --t)
                        dx[ot] = mfma_bf16(wf, __builtin_bit_cast(bf16x8, make_uint4(dut[s][t][0], dut[s][t][1], dut[s][t][2], dut[s][t][3])), dx[ot]);
                }
        }
        a0 = a1;
        a1 = a2;
        a2 = a3;
    }
}

// Waits for a load here, on every path.  (The compiler waits where a value is used, for as many requests as can be in flight there on the path
// with the fewest: behind a conditional load or store that is for all of them, the next tile's data or this tile's stores among them.)
template <typename T, int N> __device__ __forceinline__ void arrived(T (&v)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(v[i]));
}
template <int ET> __device__ __forceinline__ void arrived(SliceDraws<ET> &D)
{
    arrived(D.noise);
    arrived(D.e);
    arrived(D.row);
    arrived(D.dp);
    arrived(D.u);
}

// Rows of the per-wavefront staging tile are 36 floats apart: 16-byte reads at a stride of one row then fall into
// distinct banks.
constexpr int kRbStageRow = 36;

// dL/dh of a tile's slices: router path dx plus the expert-path rows of their k assignments, one rounding.  The rows are
// gathered and the result is stored through a tile of LDS private to the wavefront (stg), one 32-feature tile at a
// time, so that every memory instruction covers whole 128-byte (gather) or 64-byte (store) runs: eight lanes per
// slice fetch and add the k row pieces, lane (j, g) picks up its accumulator order from the tile, adds the router
// path, rounds, and puts the packed row back for four lanes per slice to store.
// A lane's part: pieces lane % 8 of the slices 8 it + lane / 8.  rows[it][jj]: their first stacked rows (negative: none), which have been
// requested (`ahead`) unless AHEAD is 0.
template <int DS, int AHEAD> struct RowsAhead {
    f32x4 v[SliceTiles<DS>::OT][4][AHEAD > 0 ? AHEAD : 1];
};
// Without a condition, which would be a branch with a wait behind it: the caller adds it only if the row is there.
template <int DS>
__device__ __forceinline__ f32x4 gradient_row_piece(const float *__restrict__ dxrow, int row, int ot, int piece)
{
    const int c = DS % 32 == 0 || 32 * ot + 4 * piece < DS ? 32 * ot + 4 * piece : 0;
    return *(const f32x4 *)(dxrow + (size_t)max(row, 0) * DS + c);
}
// The stacked rows of the first assignments of the slices whose pieces a lane handles (of others where there are none: see assemble_rows).
__device__ __forceinline__ void slice_rows(int (&rows)[4][kRbAhead], const int32_t *__restrict__ inv, long long n0, long long Ns, int k, int lane)
{
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const long long ns = n0 + it * 8 + (lane >> 3);
#pragma unroll
        for (int jj = 0; jj < kRbAhead; ++jj) rows[it][jj] = inv[min(ns, Ns - 1) * k + min(jj, k - 1)];
    }
}
// FULL: every slice of the tile exists (stores without a condition: their number in flight is known, and a wait for later loads
// is not one for them).  TOGETHER: the eight pieces of a feature tile are requested together, not two by two.
template <int DS, int AHEAD, int SROWS, bool TOGETHER, bool FULL>
__device__ __forceinline__ void assemble_rows_of(const f32x16 (&dx)[SliceTiles<DS>::OT], const int (&rows)[4][kRbAhead], const RowsAhead<DS, AHEAD> &ahead,
                                              const float *__restrict__ dxrow, const int32_t *__restrict__ inv, int k, bf16_t *__restrict__ dh,
                                              long long n0, long long Ns, int lane, float *stg)
{
    constexpr int OT = SliceTiles<DS>::OT;
    const int j = lane & 31, g = lane >> 5, piece = lane & 7, sl = lane >> 3;
#pragma unroll
    for (int ot = 0; ot < OT; ++ot) {
        f32x4 got[4][kRbAhead];
        if constexpr (TOGETHER) {
#pragma unroll
            for (int it = 0; it < 4; ++it)
#pragma unroll
                for (int jj = 0; jj < kRbAhead; ++jj) got[it][jj] = gradient_row_piece<DS>(dxrow, rows[it][jj], ot, piece);
        }
#pragma unroll
        for (int s0 = 0; s0 < 32; s0 += SROWS) {
#pragma unroll
            for (int it = s0 / 8; it < (s0 + SROWS) / 8; ++it) {
                f32x4 v = {0.f, 0.f, 0.f, 0.f};
                const long long ns = n0 + it * 8 + sl;
#pragma unroll
                for (int jj = 0; jj < kRbAhead; ++jj) {
                    f32x4 t;
                    if constexpr (AHEAD > 0) t = ahead.v[ot][it][jj];
                    else if constexpr (TOGETHER) t = got[it][jj];
                    else t = gradient_row_piece<DS>(dxrow, rows[it][jj], ot, piece);
                    const bool there = jj < k && (FULL || ns < Ns) && rows[it][jj] >= 0;
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[c] += there ? t[c] : 0.f;
                }
                for (int jj = kRbAhead; jj < k; ++jj) {
                    const int row = FULL || ns < Ns ? inv[ns * k + jj] : -1;
                    const f32x4 t = gradient_row_piece<DS>(dxrow, row, ot, piece);
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[c] += row >= 0 ? t[c] : 0.f;
                }
                *(f32x4 *)(stg + (it * 8 + sl - s0) * kRbStageRow + 4 * piece) = v;
            }
            wave_lds_sync();
            uint2 o[4];
            if (SROWS == 32 || (j & ~(SROWS - 1)) == s0) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 t = *(const f32x4 *)(stg + (j - s0) * kRbStageRow + 8 * q + 4 * g);
                    o[q] = make_uint2(pack_bf16x2(dx[ot][4 * q] + t[0], dx[ot][4 * q + 1] + t[1]),
                                      pack_bf16x2(dx[ot][4 * q + 2] + t[2], dx[ot][4 * q + 3] + t[3]));
                }
            }
            wave_lds_sync();   // every lane has read its sums: the tile now takes the packed rows (64 bytes per slice)
            if (SROWS == 32 || (j & ~(SROWS - 1)) == s0) {
#pragma unroll
                for (int q = 0; q < 4; ++q) *(uint2 *)((char *)(stg + (j - s0) * kRbStageRow) + (8 * q + 4 * g) * 2) = o[q];
            }
            wave_lds_sync();
#pragma unroll
            for (int half = 0; half < SROWS / 16; ++half) {
                const int i = half * 16 + (lane >> 2), pc = lane & 3;
                const long long ns = n0 + s0 + i;
                if ((FULL || ns < Ns) && (DS % 32 == 0 || 32 * ot + 8 * pc < DS))
                    *(uint4 *)(dh + ns * DS + 32 * ot + 8 * pc) = *(const uint4 *)((const char *)(stg + i * kRbStageRow) + pc * 16);
            }
            wave_lds_sync();   // before the next gather overwrites the tile
        }
    }
}
template <int DS, int AHEAD, int SROWS, bool TOGETHER>
__device__ __forceinline__ void assemble_rows(const f32x16 (&dx)[SliceTiles<DS>::OT], const int (&rows)[4][kRbAhead], const RowsAhead<DS, AHEAD> &ahead,
                                              const float *__restrict__ dxrow, const int32_t *__restrict__ inv, int k, bf16_t *__restrict__ dh,
                                              long long n0, long long Ns, int lane, float *stg)
{
    if (TOGETHER && n0 + 32 <= Ns) assemble_rows_of<DS, AHEAD, SROWS, TOGETHER, true>(dx, rows, ahead, dxrow, inv, k, dh, n0, Ns, lane, stg);
    else assemble_rows_of<DS, AHEAD, SROWS, TOGETHER, false>(dx, rows, ahead, dxrow, inv, k, dh, n0, Ns, lane, stg);
}


// ------------------------------------------------------------------------------------------------ logits kernel
// LDS: w1f | w2f | b1 | b2 (the first, second, sixth and seventh pieces of the packed buffer).
template <int DS, int ET>
__global__ __launch_bounds__(kRbThreads) void bwd_route_logits_mfma_kernel(
    const bf16_t *__restrict__ x, long long Ns, int E, int k, const char *__restrict__ packed, RouterBwdPacked L,
    const float *__restrict__ noise, float sigma, float inv_tau, const float *__restrict__ drop_u, float rate,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ inv, const float *__restrict__ dpk,
    CapLoss cap, bf16_t *__restrict__ dg_terms /* [terms][Ns][EP] */, uint32_t *__restrict__ relu_bits)
{
    constexpr int KS = SliceTiles<DS>::KS, EP = ET * 32, TERMS = kRbTerms<DS>;
    extern __shared__ __align__(16) char lds[];
    uint4 *w1f = (uint4 *)lds;                              // [8][KS][64]
    uint4 *w2f = w1f + kRbHT * KS * 64;                     // [8][2][ET][64]
    float *b1s = (float *)(w2f + ET * kRbHT * 2 * 64);      // [256]
    float *b2s = b1s + kRbHr;                               // [EP]
    __shared__ unsigned long long cap_part[kRbWaves * 64];
    __shared__ float capg_s[64];

    const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (cap.slots != nullptr) capacity_part<kRbWaves>(cap, E, tid, cap_part);
    stage_bytes(packed + L.w1f, (char *)w1f, (size_t)kRbHT * KS * 1024, tid, kRbThreads);
    stage_bytes(packed + L.w2f, (char *)w2f, (size_t)ET * kRbHT * 2 * 1024, tid, kRbThreads);
    if (tid < kRbHr) b1s[tid] = ((const float *)(packed + L.b1))[tid];
    if (tid < EP) b2s[tid] = ((const float *)(packed + L.b2))[tid];
    __syncthreads();
    if (cap.slots != nullptr) {
        capacity_derivatives<kRbWaves>(cap, E, tid, cap_part, capg_s);
        __syncthreads();
    }

    const long long ntiles = (Ns + 31) / 32;
    for (long long tile = (long long)wave * gridDim.x + blockIdx.x; tile < ntiles; tile += (long long)gridDim.x * kRbWaves) {
        const long long n = tile * 32 + j;
        const bool valid = n < Ns;
        const long long nn = valid ? n : 0;   // a lane without a slice reads slice 0 and writes nothing
        const uint4 *xr = (const uint4 *)(x + nn * DS);
        bf16x8 xb[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) xb[ks] = load_row_piece<DS>(xr, ks, g);
        f32x16 gacc[ET];
        uint32_t act[4], dgt[ET][TERMS][8];
        router_logits<DS, ET>(xb, w1f, w2f, b1s, b2s, lane, g, gacc, act);
        SliceDraws<ET> D;
        load_draws<ET>(D, nn, g, E, k, noise, drop_u, idx, inv, dpk);
        logit_gradients<ET, TERMS>(gacc, D, nn, g, E, k, noise != nullptr, sigma, inv_tau, drop_u, rate, idx, inv, dpk, cap.slots != nullptr, capg_s, dgt);
        if (valid) {
            store_logit_gradients<ET, TERMS>(dgt, dg_terms, Ns, n, g);
            *(uint4 *)(relu_bits + (n * 2 + g) * 4) = make_uint4(act[0], act[1], act[2], act[3]);
        }
    }
}

// ------------------------------------------------------------------------------------------------ inputs kernel
// LDS: w2c | w1c (the third and fourth pieces of the packed buffer, adjacent) | staging tiles.
// Bound: memory, 0.8 GB at width 128, 64 experts, 524 288 slices: 208 us.  With the gradient rows of a feature tile requested together
// it takes 181 alone, but runs beside the expert weight gradients, and the whole backward is slower by 3% (2.50 / 2.60 ms).
template <int DS, int ET>
__global__ __launch_bounds__(kRbThreads) void bwd_route_inputs_mfma_kernel(
    long long Ns, int k, const char *__restrict__ packed, RouterBwdPacked L, const int32_t *__restrict__ inv,
    const float *__restrict__ dxrow, const bf16_t *__restrict__ dg_terms, const uint32_t *__restrict__ relu_bits,
    bf16_t *__restrict__ dh)
{
    constexpr int OT = SliceTiles<DS>::OT, EP = ET * 32, TERMS = kRbTerms<DS>;
    extern __shared__ __align__(16) char lds[];
    const uint4 *w2c = (const uint4 *)lds;                       // [ET][2][8][64]
    const uint4 *w1c = w2c + ET * 2 * kRbHT * 64;                // [8][2][OT][64]
    float *stg_all = (float *)(w1c + kRbHT * 2 * OT * 64);       // [8 wavefronts][32][kRbStageRow]

    const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    stage_bytes(packed + L.w2c, lds, (size_t)(ET * 2 * kRbHT + kRbHT * 2 * OT) * 1024, tid, kRbThreads);
    __syncthreads();
    float *stg = stg_all + wave * 32 * kRbStageRow;

    const long long ntiles = (Ns + 31) / 32;
    for (long long tile = (long long)wave * gridDim.x + blockIdx.x; tile < ntiles; tile += (long long)gridDim.x * kRbWaves) {
        const long long n = tile * 32 + j;
        const bool valid = n < Ns;
        // dL/dg of this lane in accumulator order: register pairs, i.e. B-operand fragments, as they were stored
        uint32_t dgt[ET][TERMS][8], act[4] = {0, 0, 0, 0};
#pragma unroll
        for (int et = 0; et < ET; ++et)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
#pragma unroll
                for (int t = 0; t < TERMS; ++t) {
                    uint2 v = make_uint2(0, 0);   // a lane without a slice contributes nothing
                    if (valid) v = *(const uint2 *)(dg_terms + (t * Ns + n) * EP + et * 32 + 8 * q + 4 * g);
                    dgt[et][t][2 * q] = v.x;
                    dgt[et][t][2 * q + 1] = v.y;
                }
            }
        if (valid) {
            const uint4 b = *(const uint4 *)(relu_bits + (n * 2 + g) * 4);
            act[0] = b.x; act[1] = b.y; act[2] = b.z; act[3] = b.w;
        }
        f32x16 dx[OT];
        input_gradients<DS, ET>(dgt, act, w2c, w1c, lane, dx);
        int rows[4][kRbAhead];
        slice_rows(rows, inv, tile * 32, Ns, k, lane);
        RowsAhead<DS, 0> none;
        assemble_rows<DS, 0, 32, false>(dx, rows, none, dxrow, inv, k, dh, tile * 32, Ns, lane, stg);
    }
}

// ------------------------------------------------------------------------------------------------ both in one
// Where the fragments of both halves fit the LDS together: dL/dg and the ReLU pattern stay in registers, x of the next tile and the
// first two gradient rows of every slice are requested ahead of the matrix instructions that they wait behind.
// Bound: the latency of two wavefronts per SIMD (33 thousand cycles per tile, of which 2340 vector and 160 matrix instructions issue in
// 11 thousand); four would not hold the gradient rows (128 registers: spills, 187 us).
// 262 144 slices at width 64, 32 experts: logits 60 + inputs 83 us -> 93 us, of which the gradient rows' loads without a branch and a
// wait behind each are 25, the ReLU pattern in two instructions per unit, the capped median and the mixed-precision split 14 (the packed
// maximum that keeps an infinity costs 1 to 3 of them).  32 768 slices at width 48: 17 + 20 -> 24 us.  Width 96, 65 528 slices: 40.8 -> 37.6
// us with the gradient rows of a feature tile requested together (assemble_rows) and no wait for the next tile's data or this one's stores;
// where they are requested ahead anyway (AHEAD) the same order of requests changes nothing.
template <int DS, int ET, int THREADS, int AHEAD, int SROWS>
__global__ __launch_bounds__(THREADS) void bwd_route_slices_mfma_kernel(
    const bf16_t *__restrict__ x, long long Ns, int E, int k, const char *__restrict__ packed, RouterBwdPacked L,
    const float *__restrict__ noise, float sigma, float inv_tau, const float *__restrict__ drop_u, float rate,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ inv, const float *__restrict__ dpk,
    CapLoss cap, const float *__restrict__ dxrow, bf16_t *__restrict__ dg_terms /* [terms][Ns][EP] */, bf16_t *__restrict__ dh)
{
    constexpr int KS = SliceTiles<DS>::KS, OT = SliceTiles<DS>::OT, EP = ET * 32, TERMS = kRbTerms<DS>, kWaves = THREADS / 64;
    constexpr bool EARLY = AHEAD == 0;   // the next tile's stacked rows with its x, both waited for in front of this tile's stores
    extern __shared__ __align__(16) char lds[];
    uint4 *w1f = (uint4 *)lds;                              // [8][KS][64]
    uint4 *w2f = w1f + kRbHT * KS * 64;                     // [8][2][ET][64]
    uint4 *w2c = w2f + ET * kRbHT * 2 * 64;                 // [ET][2][8][64]
    uint4 *w1c = w2c + ET * 2 * kRbHT * 64;                 // [8][2][OT][64]
    float *b1s = (float *)(w1c + kRbHT * 2 * OT * 64);      // [256]
    float *b2s = b1s + kRbHr;                               // [EP]
    float *capg_s = b2s + EP;                               // [64]
    float *stg_all = capg_s + 64;                           // [wavefronts][SROWS][kRbStageRow]; first the capacity sums' parts [wavefronts][64]

    const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *stg = stg_all + wave * SROWS * kRbStageRow;
    // A block takes consecutive tiles: the gradient rows of a run of slices are runs of rows in every expert, on few memory pages.
    const long long all = (Ns + 31) / 32, per = (all + gridDim.x - 1) / gridDim.x, ntiles = min(all, (blockIdx.x + 1) * per), step = kWaves;
    long long tile = blockIdx.x * per + wave;

    auto load_x = [&](long long t, bf16x8 (&xb)[KS]) {   // a lane without a slice reads slice 0 and writes nothing
        const long long n = t * 32 + j;
        const uint4 *xr = (const uint4 *)(x + (n < Ns ? n : 0) * DS);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) xb[ks] = load_row_piece<DS>(xr, ks, g);
    };
    bf16x8 xb[KS];
    int rows[4][kRbAhead];
    load_x(tile, xb);
    slice_rows(rows, inv, tile * 32, Ns, k, lane);
    if (cap.slots != nullptr) capacity_part<kWaves>(cap, E, tid, (unsigned long long *)stg_all);
    stage_bytes(packed + L.w1f, (char *)w1f, (size_t)(kRbHT * KS + ET * kRbHT * 2 + ET * 2 * kRbHT + kRbHT * 2 * OT) * 1024, tid, THREADS);   // (adjacent)
    if (tid < kRbHr) b1s[tid] = ((const float *)(packed + L.b1))[tid];
    if (tid < EP) b2s[tid] = ((const float *)(packed + L.b2))[tid];
    __syncthreads();
    if (cap.slots != nullptr) {
        capacity_derivatives<kWaves>(cap, E, tid, (const unsigned long long *)stg_all, capg_s);
        __syncthreads();
    }

    for (; tile < ntiles; tile += step) {
        const long long n = tile * 32 + j, nn = n < Ns ? n : 0;
        SliceDraws<ET> D;
        RowsAhead<DS, AHEAD> ahead;
        if constexpr (AHEAD > 0) {
#pragma unroll
            for (int ot = 0; ot < OT; ++ot)
#pragma unroll
                for (int it = 0; it < 4; ++it)
#pragma unroll
                    for (int jj = 0; jj < AHEAD; ++jj) ahead.v[ot][it][jj] = gradient_row_piece<DS>(dxrow, rows[it][jj], ot, lane & 7);
        }
        load_draws<ET>(D, nn, g, E, k, noise, drop_u, idx, inv, dpk);
        f32x16 gacc[ET], dx[OT];
        uint32_t act[4], dgt[ET][TERMS][8];
        router_logits<DS, ET>(xb, w1f, w2f, b1s, b2s, lane, g, gacc, act);
        if constexpr (EARLY) arrived(D);
        int next[4][kRbAhead];
        load_x(tile + step, xb);
        if (EARLY) slice_rows(next, inv, (tile + step) * 32, Ns, k, lane);
        logit_gradients<ET, TERMS>(gacc, D, nn, g, E, k, noise != nullptr, sigma, inv_tau, drop_u, rate, idx, inv, dpk, cap.slots != nullptr, capg_s, dgt);
        if constexpr (EARLY) {
            arrived(xb);
#pragma unroll
            for (int it = 0; it < 4; ++it) arrived(next[it]);
        }
        if (n < Ns) store_logit_gradients<ET, TERMS>(dgt, dg_terms, Ns, n, g);
        input_gradients<DS, ET>(dgt, act, w2c, w1c, lane, dx);
        if (!EARLY) slice_rows(next, inv, (tile + step) * 32, Ns, k, lane);
        assemble_rows<DS, AHEAD, SROWS, EARLY>(dx, rows, ahead, dxrow, inv, k, dh, tile * 32, Ns, lane, stg);
#pragma unroll
        for (int it = 0; it < 4; ++it)
#pragma unroll
            for (int jj = 0; jj < kRbAhead; ++jj) rows[it][jj] = next[it][jj];
    }
}

// ----------------------------------------------------------------------------------------------- weights kernel
// The transposed layout: a block of eight wavefronts, one per hidden tile, walks 32-slice units.  x and the dL/dg terms of a
// unit (contiguous rows of the tables) are loaded a unit ahead and put into one of two LDS buffers in front of the one barrier
// per unit; as A operands they give u^T and dL/du^T (lane = hidden unit, registers = slices), and read back transposed they are
// the other operand of dWr1 += x^T dL/du and dWr2 += u^T dL/dg, whose own operand comes from those registers.
// Bound: the matrix pipe nominally (22 instructions per tile and unit at width 64, 32 experts).  262 144 slices at that
// shape, with the transposes in the LDS instead of on the matrix pipe and rows loaded ahead: 95 -> 60 us; 524 288
// slices at width 128, 64 experts: 405 -> 166 us.  At width 48 (32 768 slices, with the logits and inputs kernels): 4.0 ms of
// vector-ALU kernel -> 52 us.
constexpr int kRbUnit = 32;
template <int DS, int ET, int TERMS> struct RouterWeightsTile {
    static constexpr int KS = SliceTiles<DS>::KS, OT = SliceTiles<DS>::OT, GS = 2 * ET;   // GS: K-steps of 16 experts
    static constexpr bool WLDS = DS >= 96;                                                 // fragments of Wr1 in LDS (else registers)
    static constexpr size_t x_bytes = (size_t)kRbUnit * LdsRows<DS>::STRIDE, g_bytes = (size_t)kRbUnit * LdsRows<32 * ET>::STRIDE;
    static constexpr size_t buf_bytes = x_bytes + TERMS * g_bytes;
    static constexpr size_t off_red = 2 * buf_bytes;                        // [2 ET][32] partial dbr2
    static constexpr size_t off_w = off_red + 2 * ET * 32 * sizeof(float);
    static constexpr size_t lds = off_w + (WLDS ? (size_t)kRbHT * KS * 1024 : 0);
};

template <int DS, int ET, int TERMS>
__global__ __launch_bounds__(kRbThreads, DS <= 128 ? 2 : 1) void bwd_route_weights_mfma_kernel(
    const bf16_t *__restrict__ x, long long Ns, int E, const char *__restrict__ packed, RouterBwdPacked L,
    const bf16_t *__restrict__ dg /* [TERMS][Ns][32 ET] */, int units_per_block, size_t slot_floats, float *__restrict__ part)
{
    typedef RouterWeightsTile<DS, ET, TERMS> G;
    typedef LdsRows<DS> XR;
    typedef LdsRows<32 * ET> GR;
    constexpr int KS = G::KS, OT = G::OT, GS = G::GS, EP = 32 * ET, PX = XR::P, PG = GR::P;
    constexpr int kPieces = kRbUnit * (PX + TERMS * PG), NX = (kPieces + kRbThreads - 1) / kRbThreads;
    extern __shared__ __align__(16) char lds[];

    const int tid = threadIdx.x, lane = tid & 63, jj = lane & 31, g = lane >> 5;
    const int ht = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long long n_begin = (long long)blockIdx.x * units_per_block * kRbUnit;   // < Ns by the launch
    const int nrows = (int)min((long long)units_per_block * kRbUnit, Ns - n_begin);

    // ---- the pieces this thread moves: source (row 0 of the block), row, step between rows, LDS offset
    const bf16_t *msrc[NX];
    int mrow[NX], mstep[NX], mdst[NX];
    bool mx[NX];
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const int q = min(tid + i * kRbThreads, kPieces - 1);
        if (q < kRbUnit * PX) {
            mrow[i] = q / PX;
            mstep[i] = DS;
            msrc[i] = x + n_begin * DS + 8 * (q % PX);
            mdst[i] = XR::offset(mrow[i], q % PX);
            mx[i] = true;
        } else {
            const int r = q - kRbUnit * PX, t = r / (kRbUnit * PG), rr = r - t * (kRbUnit * PG);
            mrow[i] = rr / PG;
            mstep[i] = EP;
            msrc[i] = dg + ((long long)t * Ns + n_begin) * EP + 8 * (rr % PG);
            mdst[i] = (int)G::x_bytes + t * (int)G::g_bytes + GR::offset(mrow[i], rr % PG);
            mx[i] = false;
        }
    }
    uint4 mv[NX];
    auto load_rows = [&](int r0) {
#pragma unroll
        for (int i = 0; i < NX; ++i) mv[i] = *(const uint4 *)(msrc[i] + (unsigned)(min(r0 + mrow[i], nrows - 1) * mstep[i]));
    };
    auto store_rows = [&](int r0, int buf) {   // dL/dg of slices past the end is zero, so they add nothing
#pragma unroll
        for (int i = 0; i < NX; ++i)
            if (NX * kRbThreads == kPieces || tid + i * kRbThreads < kPieces)
                *(uint4 *)(lds + buf * G::buf_bytes + mdst[i]) = mx[i] || r0 + mrow[i] < nrows ? mv[i] : make_uint4(0, 0, 0, 0);
    };
    // ---- fragment addresses: rows as A operand, and transposed
    const int ax = jj * XR::STRIDE + ((g ^ XR::swizzle(jj)) << 4), ag = jj * GR::STRIDE + ((g ^ GR::swizzle(jj)) << 4);
    const int c16 = lane & 15, G4 = lane >> 4, trow = 4 * g + (c16 >> 2), tpiece = 2 * (G4 & 1) + ((lane & 3) >> 1);
    const int tx = trow * XR::STRIDE + ((tpiece ^ XR::swizzle(trow)) << 4) + 8 * (lane & 1);
    const int tg = trow * GR::STRIDE + ((tpiece ^ GR::swizzle(trow)) << 4) + 8 * (lane & 1);
    auto transposed = [&](const char *rows, int base, int stride, int tile, int s) {   // rows 16 s .., columns 32 tile ..
        const char *p = rows + 16 * s * stride + (base ^ (tile << 6));
        return read_transposed(as_lds(p), as_lds(rows + (16 * s + 8) * stride + (base ^ (tile << 6) ^ 32)));
    };

    load_rows(0);
    // ---- this wavefront's weights
    bf16x8 w1r[G::WLDS ? 1 : KS], w2r[GS];
    if constexpr (G::WLDS) {
        stage_bytes(packed + L.w1f, lds + G::off_w, (size_t)kRbHT * KS * 1024, tid, kRbThreads);
    } else {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) w1r[ks] = __builtin_bit_cast(bf16x8, ((const uint4 *)(packed + L.w1f))[(ht * KS + ks) * 64 + lane]);
    }
#pragma unroll
    for (int s = 0; s < GS; ++s) w2r[s] = __builtin_bit_cast(bf16x8, ((const uint4 *)(packed + L.w2r))[(ht * GS + s) * 64 + lane]);
    const float bias = ((const float *)(packed + L.b1))[ht * 32 + jj];
    if constexpr (XR::PW > PX) {   // the pieces past the slice width stay zero
        for (int t = tid; t < 2 * kRbUnit * (XR::PW - PX); t += kRbThreads) {
            const int row = t / (XR::PW - PX), piece = PX + t % (XR::PW - PX);
            *(uint4 *)(lds + (row / kRbUnit) * G::buf_bytes + XR::offset(row % kRbUnit, piece)) = make_uint4(0, 0, 0, 0);
        }
    }
    store_rows(0, 0);
    __syncthreads();

    // dWr2 and dbr2 with three terms: the products of small terms are summed on their own, so that the large ones are rounded as
    // seldom as there are K-steps
    f32x16 aW1[OT], aW2[ET], aW2s[ET];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
#pragma unroll
        for (int et = 0; et < ET; ++et) aW2[et][i] = aW2s[et][i] = 0.f;
#pragma unroll
        for (int ot = 0; ot < OT; ++ot) aW1[ot][i] = 0.f;
    }
    float ab1 = 0.f, ab2 = 0.f, ab2s = 0.f;
    int buf = 0;
#pragma unroll 1
    for (int r0 = 0; r0 < nrows; r0 += kRbUnit) {
        const bool more = r0 + kRbUnit < nrows;
        if (more) load_rows(r0 + kRbUnit);
        const char *xs = lds + buf * G::buf_bytes, *gs = xs + G::x_bytes;
        f32x16 u, du;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            u[i] = bias;
            du[i] = 0.f;
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 wf = G::WLDS ? __builtin_bit_cast(bf16x8, ((const uint4 *)(lds + G::off_w))[(ht * KS + ks) * 64 + lane]) : w1r[G::WLDS ? 0 : ks];
            u = mfma_bf16(*(const bf16x8 *)(xs + (ax ^ (ks << 5))), wf, u);
        }
        // A matrix instruction whose products outweigh its accumulator input cuts the latter off toward minus infinity, which adds
        // up in dbr1: so the large term comes first, and with three terms every K-step starts from zero.
#pragma unroll
        for (int s = 0; s < GS; ++s) {
            const bool fresh = TERMS == 3 && s > 0;
            f32x16 d;
#pragma unroll
            for (int i = 0; i < 16; ++i) d[i] = fresh ? 0.f : du[i];
#pragma unroll
            for (int t = 0; t < TERMS; ++t) d = mfma_bf16(*(const bf16x8 *)(gs + t * G::g_bytes + (ag ^ (s << 5))), w2r[s], d);
#pragma unroll
            for (int i = 0; i < 16; ++i) du[i] = fresh ? du[i] + d[i] : d[i];
        }
        uint32_t up[2][TERMS][4], dup[2][TERMS][4];   // by half of the unit (K-step)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float uv[4], dv[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                dv[c] = u[4 * q + c] > 0.f ? du[4 * q + c] : 0.f;
                uv[c] = fmaxf(u[4 * q + c], 0.f);
            }
            ab1 += (dv[0] + dv[1]) + (dv[2] + dv[3]);
            split_terms<TERMS>(uv, up[q >> 1], 2 * (q & 1));
            split_terms<TERMS>(dv, dup[q >> 1], 2 * (q & 1));
        }
        auto frag = [](const uint32_t (&v)[4]) { return __builtin_bit_cast(bf16x8, make_uint4(v[0], v[1], v[2], v[3])); };
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int et = 0; et < ET; ++et) {   // dWr2 [hidden unit][expert]: lane = expert; small products first
                bf16x8 gt[TERMS];
#pragma unroll
                for (int t = 0; t < TERMS; ++t) gt[t] = transposed(gs + t * G::g_bytes, tg, GR::STRIDE, et, s);
#pragma unroll
                for (int o = TERMS == 3 ? 4 : 1; o >= 0; --o)   // two terms: products down to the second's size
#pragma unroll
                    for (int t = 0; t < TERMS; ++t)
                        if (o - t >= 0 && o - t < TERMS) {
                            if (TERMS == 3 && o > 0) aW2s[et] = mfma_bf16(frag(up[s][o - t]), gt[t], aW2s[et]);
                            else aW2[et] = mfma_bf16(frag(up[s][o - t]), gt[t], aW2[et]);
                        }
                if (ht == 2 * et + s) {   // dbr2: the sums of dL/dg over the slices, one fragment per wavefront
#pragma unroll
                    for (int t = TERMS - 1; t > 0; --t) ab2s += fragment_sum(gt[t]);
                    ab2 += fragment_sum(gt[0]);
                }
            }
#pragma unroll
            for (int ot = 0; ot < OT; ++ot) {   // dWr1 [slice feature][hidden unit]: lane = hidden unit
                const bf16x8 xt = transposed(xs, tx, XR::STRIDE, ot, s);
#pragma unroll
                for (int t = TERMS - 1; t >= 0; --t) aW1[ot] = mfma_bf16(xt, frag(dup[s][t]), aW1[ot]);
            }
        }
        if (more) store_rows(r0 + kRbUnit, buf ^ 1);
        lds_barrier();
        buf ^= 1;
    }

    // ---- this block's slot: dWr1 [ds][Hr] | dWr2 [Hr][E] | dbr1 [Hr] | dbr2 [E]
    if constexpr (TERMS == 3) {
#pragma unroll
        for (int et = 0; et < ET; ++et) aW2[et] += aW2s[et];
    }
    ab2 += ab2s;
    float *slot = part + (size_t)blockIdx.x * slot_floats;
    float *pWr1 = slot, *pWr2 = pWr1 + (size_t)DS * kRbHr, *pbr1 = pWr2 + (size_t)kRbHr * E, *pbr2 = pbr1 + kRbHr;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
#pragma unroll
        for (int ot = 0; ot < OT; ++ot) {
            const int f = 32 * ot + acc_feature(i, g);
            if (DS % 32 == 0 || f < DS) pWr1[(size_t)f * kRbHr + 32 * ht + jj] = aW1[ot][i];
        }
#pragma unroll
        for (int et = 0; et < ET; ++et)
            if (32 * et + jj < E) pWr2[(size_t)(32 * ht + acc_feature(i, g)) * E + 32 * et + jj] = aW2[et][i];
    }
    ab1 += __shfl_xor(ab1, 32);   // the two lane groups hold different slices of the same hidden unit
    if (g == 0) pbr1[32 * ht + jj] = ab1;
    float *red = (float *)(lds + G::off_red);
    ab2 += __shfl_xor(ab2, 32);
    if (ht < 2 * ET && g == 0) red[ht * 32 + jj] = ab2;   // [et][half of the unit][32]
    __syncthreads();
    if (tid < E) pbr2[tid] = red[(tid >> 5) * 64 + (tid & 31)] + red[(tid >> 5) * 64 + 32 + (tid & 31)];
}

// ------------------------------------------------------------------------------------------------------ host
static size_t logits_lds(int KS, int ET) { return (size_t)(kRbHT * KS + kRbHT * 2 * ET) * 1024 + (kRbHr + 32 * ET) * sizeof(float); }
static size_t inputs_lds(int OT, int ET)
{
    return (size_t)(ET * 2 * kRbHT + kRbHT * 2 * OT) * 1024 + (size_t)kRbWaves * 32 * kRbStageRow * sizeof(float);
}

// One kernel for the logits and the inputs: wavefronts per block (0: the fragments of both do not fit the LDS), gradient rows
// requested ahead, staging rows.  The rows are requested ahead where the registers hold them: 32 per output tile beside 8 per term and expert tile
// of dL/dg, in 256.  Backward in us, ahead / where they are added, k = 2, 262 144 slices: width 64, E = 32 359 / 380; width 24, E = 16 277 / 279, E = 64
// 364 / 371; width 48, E = 16 541 / 553, but E = 64 (56 registers spilled) 712 / 694, 2000 slices 89.0 / 87.3.
template <int DS, int ET> struct RouterFused {
    static constexpr size_t weights = (size_t)(kRbHT * SliceTiles<DS>::KS + 4 * ET * kRbHT + kRbHT * 2 * SliceTiles<DS>::OT) * 1024 + (kRbHr + 32 * ET + 64) * 4;
    static constexpr size_t row = (size_t)kRbStageRow * 4;
    static constexpr int SROWS = weights + 8 * 32 * row <= 160 * 1024 ? 32 : 16;
    static constexpr int AHEAD = SROWS == 32 && 32 * SliceTiles<DS>::OT + 8 * ET * kRbTerms<DS> <= 96 ? kRbAhead : 0;   // (no registers for them at the wider shapes)
    static constexpr int waves = weights + 8 * SROWS * row <= 160 * 1024 ? 8 : 0;
    static constexpr size_t lds = weights + waves * SROWS * row;
};

template <int DS> static bool router_fused_width(int ET) { return ET == 1 ? RouterFused<DS, 1>::waves > 0 : RouterFused<DS, 2>::waves > 0; }
static bool router_fused(int ds, int ET)
{
    switch (ds) {
    case 24: return router_fused_width<24>(ET);
    case 48: return router_fused_width<48>(ET);
    case 64: return router_fused_width<64>(ET);
    case 96: return router_fused_width<96>(ET);
    case 128: return router_fused_width<128>(ET);
    default: return router_fused_width<192>(ET);
    }
}

bool backward_router_mfma_shape(const slicemoe_config &c)
{
    const int ds = c.d / c.S, ET = (c.E + 31) / 32, KS = (ds + 15) / 16, OT = (ds + 31) / 32;
    return c.dtype == SLICEMOE_BF16 && (ds == 24 || ds == 48 || ds == 64 || ds == 96 || ds == 128 || ds == 192) && c.Hr == kRbHr &&
           c.E <= 64 && !(c.flags & SLICEMOE_FLAG_FORCE_GENERIC) && logits_lds(KS, ET) <= (size_t)max_lds_per_block() &&
           inputs_lds(OT, ET) <= (size_t)max_lds_per_block();
}

// scratch: the repacked router | dL/dg terms [terms][Ns][32 ET] bf16 | ReLU bits [Ns][2][4] words (between two kernels only)
struct RouterBwdScratch {
    size_t dg, bits, total;
};
static RouterBwdScratch router_bwd_scratch(const slicemoe_config &c)
{
    const size_t Ns = (size_t)c.T * c.S, ET = (size_t)(c.E + 31) / 32;
    RouterBwdScratch R;
    size_t at = align_up(router_bwd_layout(c.d / c.S, (int)ET).total, 256);
    R.dg = at;     at += align_up(backward_terms(c.d / c.S) * Ns * 32 * ET * sizeof(bf16_t), 256);
    R.bits = at;   at += router_fused(c.d / c.S, (int)ET) ? 0 : align_up(Ns * 8 * sizeof(uint32_t), 256);
    R.total = at;
    return R;
}

size_t backward_router_mfma_scratch_bytes(const slicemoe_config &c)
{
    return router_bwd_scratch(c).total;
}

// Units of 32 slices per block of the weights kernel: one block per CU, at least two units each (a block leaves a slot of
// partial sums behind, as large as the router's weights).
constexpr int kRbLeastUnits = 2;
static int router_units_per_block(const slicemoe_config &c)
{
    const long long units = ((long long)c.T * c.S + kRbUnit - 1) / kRbUnit;
    const long long per = (units + num_compute_units() - 1) / num_compute_units();
    return per < kRbLeastUnits ? kRbLeastUnits : (int)per;
}

long long backward_router_mfma_slots(const slicemoe_config &c)
{
    const long long units = ((long long)c.T * c.S + kRbUnit - 1) / kRbUnit, per = router_units_per_block(c);
    return (units + per - 1) / per;
}

long long backward_router_mfma_slots_bound(const slicemoe_config &c)
{
    const long long units = ((long long)c.T * c.S + kRbUnit - 1) / kRbUnit, most = (units + kRbLeastUnits - 1) / kRbLeastUnits;
    return most < num_compute_units() ? most : num_compute_units();
}

template <int DS, int ET>
static hipError_t run_router_mfma(const slicemoe_config &c, const RouterBwdPacked &L, const void *h, const RouteVariant &v,
                                  const float *drop_u, float rate, const int32_t *idx, const int32_t *inv, const float *dpk,
                                  const float *dxrow, void *d_h, const char *pb, bf16_t *dg, uint32_t *bits, size_t slot_floats,
                                  float *part, hipStream_t s)
{
    constexpr int KS = SliceTiles<DS>::KS, OT = SliceTiles<DS>::OT;
    const long long Ns = (long long)c.T * c.S;
    const long long ntiles = (Ns + 31) / 32, units = (ntiles + kRbWaves - 1) / kRbWaves;
    hipError_t e;
    const CapLoss cap = {v.cap_slots, (short)v.cap_nslots, (short)v.cap_bits, v.cap_alpha};
    typedef RouterFused<DS, ET> F;
    if constexpr (F::waves > 0) {
        auto fk = bwd_route_slices_mfma_kernel<DS, ET, F::waves * 64, F::AHEAD, F::SROWS>;
        if ((e = grant_dynamic_lds((const void *)fk, F::lds)) != hipSuccess) return e;
        const long long blocks = num_compute_units() < ntiles ? num_compute_units() : ntiles;   // (a small batch spreads over all CUs)
        fk<<<(int)blocks, F::waves * 64, F::lds, s>>>((const bf16_t *)h, Ns, c.E, c.k, pb, L, v.sigma > 0.f ? v.noise : nullptr, v.sigma, v.inv_tau,
                                                      rate > 0.f ? drop_u : nullptr, rate, idx, inv, dpk, cap, dxrow, dg, (bf16_t *)d_h);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else {
        auto lk = bwd_route_logits_mfma_kernel<DS, ET>;
        e = grant_dynamic_lds((const void *)lk, logits_lds(KS, ET));
        if (e != hipSuccess) return e;
        // as many blocks as can be resident at once (registers and LDS allow two per CU for the narrow shapes)
        static int lk_per_cu = 0;   // per instantiation; the same on every device of the machine
        if (lk_per_cu == 0) {
            int n = 1;
            if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void *)lk, kRbThreads, logits_lds(KS, ET))) != hipSuccess) return e;
            lk_per_cu = n < 1 ? 1 : n;
        }
        long long blocks = (long long)num_compute_units() * lk_per_cu;
        if (blocks > units) blocks = units;
        lk<<<(int)blocks, kRbThreads, logits_lds(KS, ET), s>>>((const bf16_t *)h, Ns, c.E, c.k, pb, L, v.sigma > 0.f ? v.noise : nullptr,
                                                               v.sigma, v.inv_tau, rate > 0.f ? drop_u : nullptr, rate, idx, inv, dpk,
                                                               cap, dg, bits);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        auto ik = bwd_route_inputs_mfma_kernel<DS, ET>;
        if ((e = grant_dynamic_lds((const void *)ik, inputs_lds(OT, ET))) != hipSuccess) return e;
        // one block per CU: this kernel waits on its row gathers, and a second resident block measured slower (cache misses)
        blocks = num_compute_units() < units ? num_compute_units() : units;
        ik<<<(int)blocks, kRbThreads, inputs_lds(OT, ET), s>>>(Ns, c.k, pb, L, inv, dxrow, dg, bits, (bf16_t *)d_h);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    typedef RouterWeightsTile<DS, ET, kRbTerms<DS>> G;
    auto wk = bwd_route_weights_mfma_kernel<DS, ET, kRbTerms<DS>>;
    if ((e = grant_dynamic_lds((const void *)wk, G::lds)) != hipSuccess) return e;
    wk<<<(unsigned)backward_router_mfma_slots(c), kRbThreads, G::lds, s>>>((const bf16_t *)h, Ns, c.E, pb, L, dg, router_units_per_block(c),
                                                                          slot_floats, part);
    return hipGetLastError();
}

void backward_router_pack_jobs(const slicemoe_config &c, const slicemoe_weights &w, void *scratch, BwdPackJobs &jobs)
{
    const int E = c.E, Hr = kRbHr, ds = c.d / c.S, ET = (E + 31) / 32, EP = 32 * ET;
    const int dsK = (ds + 15) / 16 * 16, dsN = (ds + 31) / 32 * 32;
    const RouterBwdPacked L = router_bwd_layout(ds, ET);
    char *pb = (char *)scratch;
    const bf16_t *Wr1 = (const bf16_t *)w.Wr1, *Wr2 = (const bf16_t *)w.Wr2;
    BwdPackJob *J = jobs.job + jobs.count;
    jobs.count += 7;
    // w1f: Wr1 [ds, Hr] itself.  w2f: Wr2 [Hr, E] with the hidden units as contraction slots, experts padded to EP.
    J[0] = bwd_pack_job(kPackLayer1, Wr1, dsK, ds, Hr, Hr, (size_t)Hr, 1, 0, pb + L.w1f, 0, 1);
    J[1] = bwd_pack_job(backward_terms(ds) == 3 ? kPackChain : kPackChainF16, Wr2, Hr, Hr, EP, E, (size_t)E, 1, 0, pb + L.w2f, 0, 1);
    // w2c: M[e][h] = Wr2[h][e] ([EP, Hr], experts as contraction slots).  w1c: M[h][c] = Wr1[c][h] ([Hr, ds]).
    J[2] = bwd_pack_job(kPackChain, Wr2, EP, E, Hr, Hr, 1, (size_t)E, 0, pb + L.w2c, 0, 1);
    J[3] = bwd_pack_job(kPackChain, Wr1, Hr, Hr, dsN, ds, 1, (size_t)Hr, 0, pb + L.w1c, 0, 1);
    // w2r: M[e][h] = Wr2[h][e] ([EP, Hr]) in plain K-steps of 16 experts
    J[4] = bwd_pack_job(kPackLayer1, Wr2, EP, E, Hr, Hr, 1, (size_t)E, 0, pb + L.w2r, 0, 1);
    J[5] = bwd_pack_job(kPackBias, w.br1, Hr, Hr, Hr, Hr, 0, 0, 0, pb + L.b1, 0, 1);
    J[6] = bwd_pack_job(kPackBias, w.br2, E, E, EP, EP, 0, 0, 0, pb + L.b2, 0, 1);
}

// scratch: backward_router_mfma_scratch_bytes, holding the repacked weights (backward_router_pack_jobs); part:
// backward_router_mfma_slots slots of slot_floats floats.  dxrow, dpk: the expert stage's row gradients and dL/dp.
hipError_t launch_backward_router_mfma(const slicemoe_config &c, const void *h,
                                       const RouteVariant &v, const float *drop_u, float rate, const int32_t *idx,
                                       const int32_t *inv, const float *dpk, const float *dxrow, void *d_h, void *scratch,
                                       size_t slot_floats, float *part, hipStream_t s)
{
    if (!backward_router_mfma_shape(c)) return hipErrorInvalidValue;
    const int ds = c.d / c.S, ET = (c.E + 31) / 32;
    const RouterBwdPacked L = router_bwd_layout(ds, ET);
    const RouterBwdScratch R = router_bwd_scratch(c);
    char *pb = (char *)scratch;
    bf16_t *dg = (bf16_t *)(pb + R.dg);
    uint32_t *bits = (uint32_t *)(pb + R.bits);
#define SLICEMOE_ROUTER_BWD(DSV)                                                                                                   \
    if (ds == DSV)                                                                                                                 \
        return ET == 1 ? run_router_mfma<DSV, 1>(c, L, h, v, drop_u, rate, idx, inv, dpk, dxrow, d_h, pb, dg, bits, slot_floats, part, s) \
                       : run_router_mfma<DSV, 2>(c, L, h, v, drop_u, rate, idx, inv, dpk, dxrow, d_h, pb, dg, bits, slot_floats, part, s);
    SLICEMOE_ROUTER_BWD(24)
    SLICEMOE_ROUTER_BWD(48)
    SLICEMOE_ROUTER_BWD(64)
    SLICEMOE_ROUTER_BWD(96)
    SLICEMOE_ROUTER_BWD(128)
    SLICEMOE_ROUTER_BWD(192)
#undef SLICEMOE_ROUTER_BWD
    return hipErrorInvalidValue;
}

}  // namespace slicemoe
