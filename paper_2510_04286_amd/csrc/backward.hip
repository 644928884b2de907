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
// Weight gradients: every block stores its partial sums in its own slot of a scratch buffer, and a second pair of
// kernels adds the slots up in a fixed order (device-wide atomic adds cost more than the arithmetic, and their order
// varies from run to run; this way the result is reproducible bit for bit).
#include <mutex>

#include "bwd_mfma.h"
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

constexpr int kRedElems = 64, kRedSeqs = 8;
// Sum of the router slots of all blocks in a fixed order: a block is 64 slot elements x 8 interleaved sequences of slots, whose
// eight partial sums are added in order at the end.
__global__ __launch_bounds__(kRedElems * kRedSeqs) void bwd_reduce_router_kernel(
    const float *__restrict__ part, int nslots, int ds, int Hr, int E,
    float *__restrict__ dWr1, float *__restrict__ dbr1, float *__restrict__ dWr2, float *__restrict__ dbr2)
{
    __shared__ float red[kRedSeqs][kRedElems];
    const int ex = threadIdx.x % kRedElems, sq = threadIdx.x / kRedElems;
    const size_t slot = router_slot_floats(ds, Hr, E);
    const size_t t = (size_t)blockIdx.x * kRedElems + ex;
    float acc = 0.f;
    if (t < slot) {
#pragma unroll 4
        for (int b = sq; b < nslots; b += kRedSeqs) acc += part[(size_t)b * slot + t];
    }
    red[sq][ex] = acc;
    __syncthreads();
    if (sq != 0 || t >= slot) return;
    acc = 0.f;
#pragma unroll
    for (int q = 0; q < kRedSeqs; ++q) acc += red[q][ex];   // fixed order
    const size_t n1 = (size_t)ds * Hr, n2 = (size_t)Hr * E;
    if (t < n1) dWr1[t] = acc;
    else if (t < n1 + n2) dWr2[t - n1] = acc;
    else if (t < n1 + n2 + Hr) dbr1[t - n1 - n2] = acc;
    else dbr2[t - n1 - n2 - Hr] = acc;
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

// Blocks of the capacity sums: two assignments per thread and up, at most one block per CU of the chip.
constexpr int kCapThreads = 1024;
static int cap_blocks(long long Na)
{
    const long long want = (Na + 2 * kCapThreads - 1) / (2 * kCapThreads);
    return (int)(want < 256 ? want : 256);
}

BackwardPlan backward_plan(const slicemoe_config &c)
{
    BackwardPlan p;
    const size_t Ns = (size_t)c.T * c.S, Na = Ns * c.k;
    const size_t ds = (size_t)(c.d / c.S);
    p.expert_slots = backward_mfma_shape(c) ? backward_weights_slots(c) : backward_generic_expert_slots(c);
    p.router_slots = backward_router_mfma_shape(c) ? backward_router_mfma_slots(c) : backward_generic_router_slots(c);
    size_t at = 0;
    p.dxrow = at;  at = align_up(at + Na * ds * sizeof(float), 256);
    p.dpk = at;    at = align_up(at + Na * sizeof(float), 256);
    p.expert_part = at;  at = align_up(at + (size_t)p.expert_slots * expert_slot_floats((int)ds, c.He) * sizeof(float), 256);
    p.router_part = at;  at = align_up(at + (size_t)p.router_slots * router_slot_floats((int)ds, c.Hr, c.E) * sizeof(float), 256);
    p.packed = at;  at = align_up(at + backward_mfma_packed_bytes(c), 256);
    p.router_scratch = at;  at = align_up(at + backward_router_mfma_scratch_bytes(c), 256);
    p.cap = at;  at = align_up(at + (size_t)c.E * (cap_blocks((long long)Na) * sizeof(unsigned long long) + sizeof(float)), 256);
    p.total = at + 256;
    return p;
}

// ---- The capacity loss (Section 3.2, Eq. 2) in its differentiable reading.  Eq. 2 is a function of integer counts;
// the router can only be trained with it (Section 3.1) through a stand-in, and the one taken here is the usual one: the
// count of expert e becomes the sum c_e of the final probabilities of the assignments routed to e, the loss
// alpha CV^2(c) with the population variance, and dL_cap/dp_a = alpha (2E / S^2) (c_e(a) - Q / S), S = sum c, Q = sum c^2.
// The sums are exact and the same on every run: each probability, a float in [0, 1], is added as the integer
// p * 2^38 (at most 2^22 * k assignments: no overflow in 64 bits; bits below 2^-38 of a tiny p are rounded off).
// Bound by launches and latency (a few hundred KiB to read): every block stores its sums in a slot of its own, which the
// one-block kernel behind it adds up, so nothing has to be cleared first; and only the router's kernels need the result,
// so the two run behind the expert rows: beside the weight gradients where those are on the other stream, else behind their
// reduction.
constexpr float kCapScale = 274877906944.f;   // 2^38

__global__ __launch_bounds__(kCapThreads) void bwd_cap_sums_kernel(const int32_t *__restrict__ idx, const float *__restrict__ pk,
                                                           long long Na, int E, unsigned long long *__restrict__ slots /* [gridDim.x][E] */)
{
    extern __shared__ unsigned long long cap_s[];
    for (int e = threadIdx.x; e < E; e += blockDim.x) cap_s[e] = 0ull;
    __syncthreads();
    for (long long a = (long long)blockIdx.x * blockDim.x + threadIdx.x; a < Na; a += (long long)gridDim.x * blockDim.x) {
        const int ee = idx[a];
        const int e = ee < 0 ? 0 : (ee >= E ? E - 1 : ee);
        const float p = fminf(fmaxf(pk[a], 0.f), 1.f);
        atomicAdd(&cap_s[e], (unsigned long long)__float2ll_rn(p * kCapScale));
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += blockDim.x) slots[(size_t)blockIdx.x * E + e] = cap_s[e];
}

// One block.  The slots' integers are added in the LDS, then every thread adds up all E sums in the same order and writes
// its experts' derivatives.
__global__ __launch_bounds__(kCapThreads) void bwd_cap_coeff_kernel(const unsigned long long *__restrict__ slots, int nslots, int E,
                                                                    float alpha, float *__restrict__ capg)
{
    extern __shared__ unsigned long long sums[];
    for (int e = threadIdx.x; e < E; e += blockDim.x) sums[e] = 0ull;
    __syncthreads();
    for (int i = threadIdx.x; i < nslots * E; i += blockDim.x) atomicAdd(&sums[i % E], slots[i]);
    __syncthreads();
    double S = 0.0, Q = 0.0;
    for (int e = 0; e < E; ++e) {
        const double c = (double)sums[e] / (double)kCapScale;
        S += c;
        Q += c * c;
    }
    for (int e = threadIdx.x; e < E; e += blockDim.x) {
        const double c = (double)sums[e] / (double)kCapScale;
        capg[e] = S > 0.0 ? (float)((double)alpha * (2.0 * E / (S * S)) * (c - Q / S)) : 0.f;
    }
}

// ---- A stream of the library's own, beside the caller's, for experts whose weight gradients are a kernel of their own (more
// hidden tiles than a block, or a width above 64).  That kernel and the reduction after it depend on nothing that the rest of
// the backward produces, and nothing but the caller depends on them, so they run on this stream while the row gradients and
// the router's kernels run on the caller's: the two chains fill each other's launch gaps and tails.  Whole backward, one
// stream / two: width 96, He 384: T = 1024 130 / 105 us, T = 8191 278 / 250; width 128, He 512: T = 1024 349 / 283,
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
    char *ws = (char *)workspace;
    RouteVariant v = v_in;
    v.capg = nullptr;
    float *dxrow = (float *)(ws + P.dxrow), *dpk = (float *)(ws + P.dpk);
    float *epart = (float *)(ws + P.expert_part), *rpart = (float *)(ws + P.router_part);

    // Both parts' repacked weights in one launch: a second one is 5-7 us of an otherwise idle stream (or waits for a free
    // CU beside the weight gradients), whatever it moves.
    BwdPackJobs jobs;
    jobs.count = 0;
    if (backward_mfma_shape(c)) backward_expert_pack_jobs(c, w, ws + P.packed, jobs);
    if (backward_router_mfma_shape(c)) backward_router_pack_jobs(c, w, ws + P.router_scratch, jobs);
    if ((e = bwd_pack_launch(jobs, s)) != hipSuccess) return e;

    const size_t eslot = expert_slot_floats(ds, c.He);
    std::unique_lock<std::mutex> side_lock(g_side_mutex, std::defer_lock);
    SideStream side = {};
    SideJoin joiner;
    hipStream_t se = s;   // stream of the expert weight gradients and their reduction
    // Where one kernel gives dL/dx and the weight gradients only their reduction could run beside the router's kernels,
    // and it takes more from the first of them than it hides (d=1024 S=16 E=32 T=16384: 13 us + 45 us in turn, 67 us
    // together, and 6 us for the fork; the whole backward 469 us on one stream, 482 us on two).
    if (backward_mfma_shape(c) && ((c.flags & SLICEMOE_FLAG_SINGLE_STREAM) || backward_weights_plan(c).fused)) {
        e = launch_backward_expert_mfma(c, h, d_out, pk, offsets, perm, ws + P.packed, eslot, dxrow, dpk, epart, s);
        if (e != hipSuccess) return e;
    } else if (backward_mfma_shape(c)) {
        side_lock.lock();
        if ((e = side_stream(&side)) != hipSuccess) return e;
        e = launch_backward_expert_mfma(c, h, d_out, pk, offsets, perm, ws + P.packed, eslot, dxrow, dpk, epart, s, &side);
        joiner.side = &side;   // from here on the side stream holds work of this call: joined on every way out
        joiner.s = s;
        se = side.stream;
        if (e != hipSuccess) return e;
    } else {
        e = launch_backward_expert_generic(c, h, w, d_out, pk, offsets, perm, eslot, dxrow, dpk, epart, s);
        if (e != hipSuccess) return e;
    }
    if ((e = launch_backward_reduce_segments(c, offsets, epart, eslot, g, se)) != hipSuccess) return e;

    if (v.cap_alpha != 0.f) {
        const int blocks = cap_blocks(Na);
        const size_t lds = (size_t)c.E * sizeof(unsigned long long);
        unsigned long long *slots = (unsigned long long *)(ws + P.cap);
        float *capg = (float *)(slots + (size_t)blocks * c.E);
        bwd_cap_sums_kernel<<<blocks, kCapThreads, lds, s>>>(idx, pk, Na, c.E, slots);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        bwd_cap_coeff_kernel<<<1, kCapThreads, lds, s>>>(slots, blocks, c.E, v.cap_alpha, capg);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        v.capg = capg;
    }

    const size_t rslot = router_slot_floats(ds, c.Hr, c.E);
    if (backward_router_mfma_shape(c)) {
        e = launch_backward_router_mfma(c, h, v, drop_u, rate, idx, inv, dpk, dxrow, d_h, ws + P.router_scratch,
                                        rslot, rpart, s);
        if (e != hipSuccess) return e;
    } else {
        e = launch_backward_router_generic(c, h, w, v, drop_u, rate, idx, inv, dpk, dxrow, d_h, rslot, rpart, s);
        if (e != hipSuccess) return e;
    }
    bwd_reduce_router_kernel<<<(unsigned)((rslot + kRedElems - 1) / kRedElems), kRedElems * kRedSeqs, 0, s>>>(rpart, (int)P.router_slots, ds, c.Hr, c.E, g.Wr1,
                                                                           g.br1, g.Wr2, g.br2);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return joiner.join();
}

}  // namespace slicemoe
