// Backward pass of the layer: gradients of a loss that depends on h and on the
// weights only through h', by the chain rule through the k-sum, the expert FFN and the Eq. 1 input weighting
// (Section 3.1), and the router (Section 3.1; temperature of Appendix B, logit noise of Section 5 and cross-slice
// dropout of Section 3.3 as in the forward).  The routing decisions -- selected experts, capacity drops, dropout
// zeroes -- are piecewise constant and held fixed; the router receives gradient through the selected probabilities,
// which weight the expert inputs: z = p (x W1) + b1, so dL/dp = sum_hidden dL/dz (x W1).
//
// Host side of it, and the small kernels every shape shares.  The expert and router parts run on the bf16 matrix-core
// kernels (backward_mfma.hip, backward_weights_mfma.hip, backward_router_mfma.hip) or, for every other shape and for fp32
// storage, on fp32 kernels (backward_generic.hip).
// Weight gradients: every block stores its partial sums in its own slot of a scratch buffer, and reduction
// kernels add the slots up in a fixed order (device-wide atomic adds cost more than the arithmetic, and their order
// varies from run to run; this way the result is reproducible bit for bit).
#include <math.h>

#include <mutex>

#include "bwd_mfma.h"
#include "capacity_scale.h"
#include "common.h"

namespace slicemoe {

__host__ __device__ __forceinline__ size_t expert_slot_floats(int ds, int He) { return 2 * (size_t)ds * He + He + ds; }
__host__ __device__ __forceinline__ size_t router_slot_floats(int ds, int Hr, int E) { return (size_t)ds * Hr + (size_t)Hr * E + Hr + E; }

__global__ void fill_zero_kernel(float *__restrict__ p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0.f;
}

static hipError_t zero_fill(float *p, size_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    const size_t want = (n + 255) / 256;
    fill_zero_kernel<<<(int)(want < 4096 ? want : 4096), 256, 0, s>>>(p, n);
    return hipGetLastError();
}

// ---- Sum of the slots, each element in a fixed order.
// Up to kReduceApartBytes of partial sums there is one launch for the router's slots and the experts' (where those are not on a
// stream of their own): a launch more costs 3-5 us of a single stream, whatever it sums.  The router's blocks come first in the
// grid: their chains are the longer ones.  Beyond, the experts' are summed at once, while they are still in a cache.  Forward and
// backward, two launches / one: width 48, He 192, 32 768 slices (37 MB): 163.9 / 160.9 us; width 64 fp32, He 256, 4000 slices
// (43 MB): 142.1 / 139.0; width 64, He 256, E 32 (63 MB): 32 208 slices 180.4 / 181.2, 262 144 slices 526.5 / 529.9.
struct ReduceArgs {
    // experts: blocks of THREADS / 4 groups of V slot elements, one expert each
    const float *epart;
    const int32_t *offsets;
    int step, overhead, blocks;
    size_t eslot;
    // router: blocks of THREADS / 8 slot elements
    const float *rpart;
    int nslots;
    size_t rslot;
    unsigned router_blocks;
    int ds, He, Hr, E;
    slicemoe_weight_grads g;
};
constexpr size_t kReduceApartBytes = (size_t)48 << 20;

// The expert's slots are vf + e .. vl + e, the blocks its steps fall into; four interleaved sequences of slots.
template <int V, int THREADS>
__device__ __forceinline__ void reduce_expert(const ReduceArgs &A, unsigned block, float *smem)
{
    typedef float vec __attribute__((ext_vector_type(V)));
    constexpr int SEQS = 4, ELEMS = THREADS / SEQS;
    vec *red = (vec *)smem;   // [SEQS][ELEMS]
    const int e = (int)(block % (unsigned)A.E), lane = threadIdx.x & 63;
    const int ex = threadIdx.x % ELEMS, sq = threadIdx.x / ELEMS;
    const size_t t = ((size_t)(block / (unsigned)A.E) * ELEMS + ex) * V;
    const RowAxis X = row_axis(A.offsets[min(lane + 1, A.E)] - A.offsets[min(lane, A.E)], A.step, A.overhead, A.blocks, lane);
    const int first = __builtin_amdgcn_readlane(X.first, e), steps = __builtin_amdgcn_readlane(X.steps, e);
    // its steps follow its overhead
    const int s0 = first + A.overhead, vf = s0 / X.share, vl = steps > 0 ? (s0 + steps - 1) / X.share : vf - 1;
    vec acc = {};
    if (t < A.eslot) {
        const float *src = A.epart + (size_t)e * A.eslot + t;
#pragma unroll 4
        for (int v = vf + sq; v <= vl; v += SEQS) acc += *(const vec *)(src + (size_t)v * A.eslot);
    }
    red[sq * ELEMS + ex] = acc;
    __syncthreads();
    if (sq != 0 || t >= A.eslot) return;
    acc = vec{};
#pragma unroll
    for (int q = 0; q < SEQS; ++q) acc += red[q * ELEMS + ex];
    const size_t nW = (size_t)A.ds * A.He;
    if (t < nW) *(vec *)(A.g.W1 + (size_t)e * nW + t) = acc;
    else if (t < 2 * nW) *(vec *)(A.g.W2 + (size_t)e * nW + (t - nW)) = acc;
    else if (t < 2 * nW + A.He) *(vec *)(A.g.b1 + (size_t)e * A.He + (t - 2 * nW)) = acc;
    else *(vec *)(A.g.b2 + (size_t)e * A.ds + (t - 2 * nW - A.He)) = acc;
}

// Eight interleaved sequences of slots.
template <int THREADS>
__device__ __forceinline__ void reduce_router(const ReduceArgs &A, unsigned block, float *red /* [SEQS][ELEMS] */)
{
    constexpr int SEQS = 8, ELEMS = THREADS / SEQS;
    const int ex = threadIdx.x % ELEMS, sq = threadIdx.x / ELEMS;
    const size_t t = (size_t)block * ELEMS + ex;
    float acc = 0.f;
    if (t < A.rslot) {
#pragma unroll 4
        for (int b = sq; b < A.nslots; b += SEQS) acc += A.rpart[(size_t)b * A.rslot + t];
    }
    red[sq * ELEMS + ex] = acc;
    __syncthreads();
    if (sq != 0 || t >= A.rslot) return;
    acc = 0.f;
#pragma unroll
    for (int q = 0; q < SEQS; ++q) acc += red[q * ELEMS + ex];
    const size_t n1 = (size_t)A.ds * A.Hr, n2 = (size_t)A.Hr * A.E;
    if (t < n1) A.g.Wr1[t] = acc;
    else if (t < n1 + n2) A.g.Wr2[t - n1] = acc;
    else if (t < n1 + n2 + A.Hr) A.g.br1[t - n1 - n2] = acc;
    else A.g.br2[t - n1 - n2 - A.Hr] = acc;
}

template <int V, int THREADS, bool EXPERTS, bool ROUTER>
__global__ __launch_bounds__(THREADS) void bwd_reduce_kernel(ReduceArgs A)
{
    __shared__ __align__(16) float smem[THREADS * (EXPERTS ? V : 1)];
    if (ROUTER && (!EXPERTS || blockIdx.x < A.router_blocks)) reduce_router<THREADS>(A, blockIdx.x, smem);
    else if (EXPERTS) reduce_expert<V, THREADS>(A, blockIdx.x - A.router_blocks, smem);
}

template <int V, int THREADS, bool EXPERTS, bool ROUTER>
static hipError_t run_reduce(ReduceArgs A, hipStream_t s)
{
    const size_t per_expert = (size_t)V * THREADS / 4, per_router = THREADS / 8;
    A.router_blocks = ROUTER ? (unsigned)((A.rslot + per_router - 1) / per_router) : 0;
    const unsigned blocks = A.router_blocks + (EXPERTS ? (unsigned)((A.eslot + per_expert - 1) / per_expert * A.E) : 0);
    bwd_reduce_kernel<V, THREADS, EXPERTS, ROUTER><<<blocks, THREADS, 0, s>>>(A);
    return hipGetLastError();
}

static hipError_t launch_reduce(const ReduceArgs &A, bool experts, bool router, hipStream_t s)
{
    const slicemoe_weight_grads &g = A.g;
    const bool vec4 = A.ds % 4 == 0 && A.He % 4 == 0 &&
                      (((uintptr_t)g.W1 | (uintptr_t)g.b1 | (uintptr_t)g.W2 | (uintptr_t)g.b2 | (uintptr_t)A.epart) & 15) == 0;
    if (!experts) return run_reduce<1, 512, false, true>(A, s);
    if (!router) return vec4 ? run_reduce<4, 256, true, false>(A, s) : run_reduce<1, 256, true, false>(A, s);
    return vec4 ? run_reduce<4, 512, true, true>(A, s) : run_reduce<1, 512, true, true>(A, s);
}

// What bounds the slice width and the router of a backward pass (the caller compares it with 60 KiB): eight rows of x and
// dL/dh', 256 hidden units of them, and eight slices of the router's layers, in fp32.
size_t backward_lds_bytes(const slicemoe_config &c)
{
    const size_t ds = (size_t)(c.d / c.S), dsp = (ds + 63) / 64 * 64;
    const size_t expert = sizeof(float) * 8 * (2 * dsp + 256);
    const size_t router = sizeof(float) * 8 * (ds + 2 * (size_t)c.Hr + 2 * (size_t)c.E);
    return expert > router ? expert : router;
}

// Blocks of the capacity sums: eight assignments per thread and up.
static int cap_blocks(long long Na)
{
    const long long want = (Na + 2047) / 2048;
    return (int)(want < kCapBlocks ? want : kCapBlocks);
}

BackwardPlan backward_plan(const slicemoe_config &c)
{
    BackwardPlan p;
    const size_t Ns = (size_t)c.T * c.S, Na = Ns * c.k;
    const size_t ds = (size_t)(c.d / c.S);
    p.expert_mfma = backward_mfma_shape(c);
    p.router_mfma = backward_router_mfma_shape(c);
    const BackwardWeightsPlan W = p.expert_mfma ? backward_weights_plan(c) : backward_generic_plan(c);
    p.expert_slots = W.slots;
    p.router_slots = p.router_mfma ? backward_router_mfma_slots(c) : backward_generic_router_slots(c);
    const size_t router_reserve = (size_t)(p.router_mfma ? backward_router_mfma_slots_bound(c) : backward_generic_router_slots_bound(c));
    size_t at = 0;
    p.dxrow = at;  at = align_up(at + Na * ds * sizeof(float), 256);
    p.dpk = at;    at = align_up(at + Na * sizeof(float), 256);
    p.expert_part = at;  at = align_up(at + (size_t)W.reserve * expert_slot_floats((int)ds, c.He) * sizeof(float), 256);
    p.router_part = at;  at = align_up(at + router_reserve * router_slot_floats((int)ds, c.Hr, c.E) * sizeof(float), 256);
    p.packed = at;  at = align_up(at + (p.expert_mfma ? backward_mfma_packed_bytes(c) : 0), 256);
    p.router_scratch = at;  at = align_up(at + (p.router_mfma ? backward_router_mfma_scratch_bytes(c) : 0), 256);
    p.cap = at;  at = align_up(at + (size_t)c.E * cap_blocks((long long)Na) * sizeof(unsigned long long), 256);
    p.total = at + 256;
    return p;
}

// ---- A stream of the library's own, beside the caller's, for experts whose weight gradients are a kernel of their own (more
// hidden tiles than a block at width 64, the widths above 96, and 96 where the one pass is slower).  That kernel and the
// reduction after it depend on nothing that the rest of the backward produces, and nothing but the caller depends on
// them, so they run on this stream while the row gradients and
// the router's kernels run on the caller's: the two chains fill each other's launch gaps and tails.  Whole backward, one
// stream / two: width 96, He 384: T = 1024 130 / 105 us; width 128, He 512: T = 1024 349 / 283,
// T = 16384 2538 / 2483; width 192, He 768: T = 1000 325 / 248, T = 4096 730 / 487; width 64, He 288: T = 16384 692 / 694.
// One stream and two events per device, made at the first such backward on
// that device and kept until the process ends; default priority, no implicit synchronisation with the null stream.
// The events are shared by all calls on a device, so the enqueueing of one call (fork .. join) holds a lock.
static std::mutex g_side_mutex;

static hipError_t side_stream(SideStream *out)
{
    static SideStream set[64];
    static bool have[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!have[dev]) {
        SideStream n = {};
        if ((e = hipStreamCreateWithFlags(&n.stream, hipStreamNonBlocking)) != hipSuccess) return e;
        if ((e = hipEventCreateWithFlags(&n.fork, hipEventDisableTiming)) != hipSuccess) return e;
        if ((e = hipEventCreateWithFlags(&n.join, hipEventDisableTiming)) != hipSuccess) return e;
        set[dev] = n;
        have[dev] = true;
    }
    *out = set[dev];
    return hipSuccess;
}

// Joins the side stream back into the caller's stream when the scope ends, on every path out of it.
struct SideJoin {
    const SideStream *side = nullptr;
    hipStream_t s = nullptr;
    hipError_t result = hipSuccess;
    ~SideJoin() { (void)join(); }
    hipError_t join()
    {
        if (side != nullptr) {
            hipError_t e = hipEventRecord(side->join, side->stream);
            if (e == hipSuccess) e = hipStreamWaitEvent(s, side->join, 0);
            if (e != hipSuccess) result = e;
            side = nullptr;
        }
        return result;
    }
};

hipError_t launch_backward(const slicemoe_config &c, const void *h, const slicemoe_weights &w, const RouteVariant &v_in,
                           const float *drop_u, float rate, const int32_t *idx, const float *pk, const int32_t *offsets,
                           const int32_t *perm, const int32_t *inv, const void *d_out, void *d_h,
                           const slicemoe_weight_grads &g, void *workspace, hipStream_t s)
{
    const long long Ns = (long long)c.T * c.S, Na = Ns * c.k;
    const int ds = c.d / c.S;
    const size_t nW = (size_t)c.E * ds * c.He;
    hipError_t e;
    if (Ns == 0) {   // nothing to sum: the gradients are zero
        if ((e = zero_fill(g.Wr1, (size_t)ds * c.Hr, s)) != hipSuccess) return e;
        if ((e = zero_fill(g.br1, (size_t)c.Hr, s)) != hipSuccess) return e;
        if ((e = zero_fill(g.Wr2, (size_t)c.Hr * c.E, s)) != hipSuccess) return e;
        if ((e = zero_fill(g.br2, (size_t)c.E, s)) != hipSuccess) return e;
        if ((e = zero_fill(g.W1, nW, s)) != hipSuccess) return e;
        if ((e = zero_fill(g.b1, (size_t)c.E * c.He, s)) != hipSuccess) return e;
        if ((e = zero_fill(g.W2, nW, s)) != hipSuccess) return e;
        return zero_fill(g.b2, (size_t)c.E * ds, s);
    }
    const BackwardPlan P = backward_plan(c);
    const BackwardWeightsPlan W = P.expert_mfma ? backward_weights_plan(c) : backward_generic_plan(c);
    char *ws = (char *)workspace;
    RouteVariant v = v_in;
    float *dxrow = (float *)(ws + P.dxrow), *dpk = (float *)(ws + P.dpk);
    float *epart = (float *)(ws + P.expert_part), *rpart = (float *)(ws + P.router_part);

    // Both parts' repacked weights in one launch: a second one is 5-7 us of an otherwise idle stream (or waits for a free
    // CU beside the weight gradients), whatever it moves.
    BwdPackJobs jobs;
    jobs.count = 0;
    if (P.expert_mfma) backward_expert_pack_jobs(c, W, w, ws + P.packed, jobs);
    if (P.router_mfma) backward_router_pack_jobs(c, w, ws + P.router_scratch, jobs);
    CapSums cap = {0, idx, pk, Na, c.E, ldexpf(1.f, capacity_fraction_bits(Na)), (unsigned long long *)(ws + P.cap)};
    if (v.cap_alpha != 0.f) {
        cap.blocks = cap_blocks(Na);
        v.cap_slots = cap.slots;
        v.cap_nslots = cap.blocks;
        v.cap_bits = capacity_fraction_bits(Na);
    }
    if ((e = bwd_pack_launch(jobs, cap, s)) != hipSuccess) return e;

    const size_t eslot = expert_slot_floats(ds, c.He);
    std::unique_lock<std::mutex> side_lock(g_side_mutex, std::defer_lock);
    SideStream side = {};
    SideJoin joiner;
    hipStream_t se = s;   // stream of the expert weight gradients and their reduction
    // Where one kernel gives dL/dx and the weight gradients only their reduction could run beside the router's kernels,
    // and it takes more from the first of them than it hides (d=1024 S=16 E=32 T=16384: 13 us + 45 us in turn, 67 us
    // together, and 6 us for the fork; the whole backward 469 us on one stream, 482 us on two).
    if (P.expert_mfma && ((c.flags & SLICEMOE_FLAG_SINGLE_STREAM) || W.fused)) {
        e = launch_backward_expert_mfma(c, W, h, d_out, pk, offsets, perm, ws + P.packed, eslot, dxrow, dpk, epart, s);
        if (e != hipSuccess) return e;
    } else if (P.expert_mfma) {
        side_lock.lock();
        if ((e = side_stream(&side)) != hipSuccess) return e;
        e = launch_backward_expert_mfma(c, W, h, d_out, pk, offsets, perm, ws + P.packed, eslot, dxrow, dpk, epart, s, &side);
        joiner.side = &side;   // from here on the side stream holds work of this call: joined on every way out
        joiner.s = s;
        se = side.stream;
        if (e != hipSuccess) return e;
    } else {
        e = launch_backward_expert_generic(c, h, w, d_out, pk, offsets, perm, eslot, dxrow, dpk, epart, s);
        if (e != hipSuccess) return e;
    }
    const size_t rslot = router_slot_floats(ds, c.Hr, c.E);
    const ReduceArgs sums = {epart, offsets, W.step, W.overhead, W.blocks, eslot, rpart, (int)P.router_slots, rslot, 0, ds, c.He, c.Hr, c.E, g};
    // the experts' slots: at once, on the stream that fills them, or together with the router's (see kReduceApartBytes)
    const bool apart = se != s || ((size_t)P.expert_slots * eslot + (size_t)P.router_slots * rslot) * sizeof(float) > kReduceApartBytes;
    if (apart && (e = launch_reduce(sums, true, false, se)) != hipSuccess) return e;

    if (P.router_mfma) {
        e = launch_backward_router_mfma(c, h, v, drop_u, rate, idx, inv, dpk, dxrow, d_h, ws + P.router_scratch,
                                        rslot, rpart, s);
        if (e != hipSuccess) return e;
    } else {
        e = launch_backward_router_generic(c, h, w, v, drop_u, rate, idx, inv, dpk, dxrow, d_h, rslot, rpart, s);
        if (e != hipSuccess) return e;
    }
    if ((e = launch_reduce(sums, !apart, true, s)) != hipSuccess) return e;
    return joiner.join();
}

}  // namespace slicemoe
