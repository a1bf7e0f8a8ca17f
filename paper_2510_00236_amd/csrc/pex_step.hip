// pex_step.hip -- the end of a training step over all tensors of a model in a few launches: squared global gradient norm, clipped
// update, moment tracking (pex_adam_step).
//
// One call per tensor and kind is three to six launches a tensor: a block of ten tensors took 40 of them and as many host calls, 150 us
// of a 350 us step on small models, whatever the sizes.  Here the tensors share the launches: a workgroup finds the tensor its
// chunk belongs to in the kernel's arguments.  Bound by HBM on large models: 20 + 8 bytes read and 12 + 8 written per parameter
// with tracking, S_id and S_sq once for both (24 + 32 bytes as two passes), and S_id once more for the norm.  Measured, ten tensors of a
// GPT-2-small block with its embedding (45.7 M parameters): update 381 us = 5.7 TB/s, what a copy reaches; norm 45 + 5; the whole
// step of the example 2052 -> 1888 us, a block of d = 128 with B=6, T=125 350 -> 148.
#include <type_traits>

#include "pex_internal.h"
#include "pex_update.h"

namespace pex {
namespace {

constexpr int GROUP = 32;                 // tensors of one launch: 2.4 KB of kernel arguments
constexpr int SUM_BLOCKS = 512;           // partial sums of squares per group of tensors, at most one more per tensor
constexpr int STEP_BLOCKS = 8192;         // workgroups of an update, at most one more per tensor

// Tensors cut into chunks of `chunk` elements (a multiple of four), one workgroup each
struct StepGroup {
    int count;
    unsigned first[GROUP + 1];
    int64_t chunk;
    pex_step_tensor t[GROUP];
    __device__ __forceinline__ int of_block(unsigned b) const
    {
        int k = 0;
        while (k + 1 < count && b >= first[k + 1]) ++k;
        return k;
    }
};

template <int WAVES>
__device__ __forceinline__ double block_sum(double s, double (&red)[WAVES])
{
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) t += red[w];
    __syncthreads();
    return t;
}

// partial[block] = sum of S_id^2 over the block's chunk
__global__ __launch_bounds__(512) void step_squares_kernel(StepGroup g, double* __restrict__ partial)
{
    const int k = g.of_block(blockIdx.x);
    const int64_t begin = (int64_t)(blockIdx.x - g.first[k]) * g.chunk, n = g.t[k].n;
    const int64_t end = begin + g.chunk < n ? begin + g.chunk : n;
    const float* x = g.t[k].S_id;
    double s = 0.0;
    for (int64_t e = begin + 4 * threadIdx.x; e + 3 < end; e += 4 * 512) {
        const float4 a = *(const float4*)(x + e);
        s += ((double)a.x * a.x + (double)a.y * a.y) + ((double)a.z * a.z + (double)a.w * a.w);
    }
    for (int64_t e = (end & ~(int64_t)3) + threadIdx.x; e < end; e += 512) s += (double)x[e] * x[e];
    __shared__ double red[8];
    s = block_sum(s, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

__global__ __launch_bounds__(1024) void step_norm_kernel(const double* __restrict__ partial, int n, double* __restrict__ sum_sq)
{
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) s += partial[i];
    __shared__ double red[16];
    s = block_sum(s, red);
    if (threadIdx.x == 0) *sum_sq = s;
}

// One chunk: the update and, with TRACK, both EMAs and partial[2 block ..] = the sums of their estimates
template <int VARIANT, bool TRACK, bool STREAM>
__global__ __launch_bounds__(256) void step_update_kernel(StepGroup g, AdamConsts c, MomentConsts mc, const double* __restrict__ sum_sq, float max_norm,
                                                          double* __restrict__ partial)
{
    clip(c, *sum_sq, max_norm);
    const int k = g.of_block(blockIdx.x);
    const pex_step_tensor t = g.t[k];
    const int64_t begin = (int64_t)(blockIdx.x - g.first[k]) * g.chunk;
    const int64_t end = begin + g.chunk < t.n ? begin + g.chunk : t.n;
    constexpr bool SQ = TRACK || VARIANT != PEX_ADAM;
    double mu2 = 0.0, sigma2 = 0.0;
    for (int64_t e = begin + 4 * threadIdx.x; e + 3 < end; e += 4 * 256) {
        auto at = [&](float* p) { return (float4*)(p + e); };
        float4 th = load4<STREAM>(at(t.theta)), m = load4<STREAM>(at(t.m)), v = load4<STREAM>(at(t.v)), a = make_float4(0.f, 0.f, 0.f, 0.f), q = a, s = a;
        const float4 i = load4<STREAM>((const float4*)(t.S_id + e));
        if (SQ) s = load4<STREAM>((const float4*)(t.S_sq + e));
        if (TRACK) { a = load4<STREAM>(at(t.ema_adam)); q = load4<STREAM>(at(t.ema_micro)); }
        adam_one<VARIANT>(th.x, m.x, v.x, i.x, s.x, c);
        adam_one<VARIANT>(th.y, m.y, v.y, i.y, s.y, c);
        adam_one<VARIANT>(th.z, m.z, v.z, i.z, s.z, c);
        adam_one<VARIANT>(th.w, m.w, v.w, i.w, s.w, c);
        store4<STREAM>(at(t.theta), th);
        store4<STREAM>(at(t.m), m);
        store4<STREAM>(at(t.v), v);
        if (TRACK) {
            moment_one(a.x, q.x, i.x, s.x, mc, mu2, sigma2);
            moment_one(a.y, q.y, i.y, s.y, mc, mu2, sigma2);
            moment_one(a.z, q.z, i.z, s.z, mc, mu2, sigma2);
            moment_one(a.w, q.w, i.w, s.w, mc, mu2, sigma2);
            store4<STREAM>(at(t.ema_adam), a);
            store4<STREAM>(at(t.ema_micro), q);
        }
    }
    for (int64_t e = (end & ~(int64_t)3) + threadIdx.x; e < end; e += 256) {      // the last tensor elements, fewer than four
        float th = t.theta[e], m = t.m[e], v = t.v[e];
        const float i = t.S_id[e], s = SQ ? t.S_sq[e] : 0.f;
        adam_one<VARIANT>(th, m, v, i, s, c);
        t.theta[e] = th;
        t.m[e] = m;
        t.v[e] = v;
        if (TRACK) {
            float a = t.ema_adam[e], q = t.ema_micro[e];
            moment_one(a, q, i, s, mc, mu2, sigma2);
            t.ema_adam[e] = a;
            t.ema_micro[e] = q;
        }
    }
    if (TRACK) {
        __shared__ double red[4];
        mu2 = block_sum(mu2, red);
        sigma2 = block_sum(sigma2, red);
        if (threadIdx.x == 0) {
            partial[2 * (int64_t)blockIdx.x] = mu2;
            partial[2 * (int64_t)blockIdx.x + 1] = sigma2;
        }
    }
}

// sums[2 k ..] of tensor k of the group from the pairs of its workgroups
__global__ __launch_bounds__(256) void step_moments_kernel(StepGroup g, const double* __restrict__ partial, double* __restrict__ sums)
{
    const int k = blockIdx.x;
    double s0 = 0.0, s1 = 0.0;
    for (unsigned i = g.first[k] + threadIdx.x; i < g.first[k + 1]; i += 256) {
        s0 += partial[2 * (int64_t)i];
        s1 += partial[2 * (int64_t)i + 1];
    }
    __shared__ double red[4];
    s0 = block_sum(s0, red);
    s1 = block_sum(s1, red);
    if (threadIdx.x == 0) {
        sums[2 * k] = s0;
        sums[2 * k + 1] = s1;
    }
}

int64_t total_elements(const pex_step_tensor* t, int count)
{
    int64_t n = 0;
    for (int k = 0; k < count; ++k) n += t[k].n;
    return n;
}

// at most `blocks` chunks and one more per tensor, of 1024 elements or more
int64_t chunk_of(int64_t n, int64_t blocks) { return ((n + blocks - 1) / blocks + 1023) / 1024 * 1024; }

StepGroup make_group(const pex_step_tensor* t, int count, int64_t chunk)
{
    StepGroup g{};
    g.count = count;
    g.chunk = chunk;
    unsigned at = 0;
    for (int k = 0; k < count; ++k) {
        g.t[k] = t[k];
        g.first[k] = at;
        at += (unsigned)((t[k].n + chunk - 1) / chunk);
    }
    g.first[count] = at;
    return g;
}

int groups_of(int count) { return (count + GROUP - 1) / GROUP; }

}  // namespace

// The workspace holds the partial sums of squares of all groups, or the pairs of one group's update.  `least`: a chunk per tensor and
// one more per group.
size_t adam_step_workspace(const pex_step_tensor* tensors, int count)
{
    size_t most = adam_step_workspace_least(count);
    const size_t squares = ((size_t)SUM_BLOCKS * groups_of(count) + (size_t)count) * sizeof(double);
    if (squares > most) most = squares;
    for (int at = 0; at < count; at += GROUP) {
        const int c = count - at < GROUP ? count - at : GROUP;
        const size_t pairs = (size_t)make_group(tensors + at, c, chunk_of(total_elements(tensors + at, c), STEP_BLOCKS)).first[c] * 2 * sizeof(double);
        if (pairs > most) most = pairs;
    }
    return most;
}

size_t adam_step_workspace_least(int count) { return ((size_t)groups_of(count) + (size_t)count) * 2 * sizeof(double); }

hipError_t launch_adam_step(const pex_step_tensor* tensors, int count, pex_adam_variant variant, const pex_adam_params& p, const pex_moment_params* track,
                            float max_norm, double* sum_sq, double* sums, void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    const AdamConsts c = adam_consts(p);
    const MomentConsts mc = track ? moment_consts(*track) : MomentConsts{};
    double* partial = (double*)workspace;
    // a smaller workspace takes fewer, larger chunks
    const int64_t room = (int64_t)(workspace_bytes / sizeof(double));
    const int64_t squares_room = (room - count) / groups_of(count), pairs_room = room / 2 - (count < GROUP ? count : GROUP);
    const int64_t sum_blocks = squares_room < SUM_BLOCKS ? squares_room : SUM_BLOCKS, step_blocks = pairs_room < STEP_BLOCKS ? pairs_room : STEP_BLOCKS;
    int nparts = 0;
    for (int at = 0; at < count; at += GROUP) {
        const int n = count - at < GROUP ? count - at : GROUP;
        const StepGroup g = make_group(tensors + at, n, chunk_of(total_elements(tensors + at, n), sum_blocks));
        step_squares_kernel<<<dim3(g.first[n]), dim3(512), 0, stream>>>(g, partial + nparts);
        nparts += (int)g.first[n];
    }
    step_norm_kernel<<<dim3(1), dim3(1024), 0, stream>>>(partial, nparts, sum_sq);
    hipError_t e = hipGetLastError();
    for (int at = 0; at < count && e == hipSuccess; at += GROUP) {
        const int n = count - at < GROUP ? count - at : GROUP;
        const int64_t elements = total_elements(tensors + at, n);
        const StepGroup g = make_group(tensors + at, n, chunk_of(elements, step_blocks));
        const bool stream_past = streams(elements, (variant == PEX_ADAM && !track ? 4 : 5) + (track ? 2 : 0));
        auto go = [&](auto kern) { kern<<<dim3(g.first[n]), dim3(256), 0, stream>>>(g, c, mc, sum_sq, max_norm, partial); };
        auto pick = [&](auto v) {
            constexpr int V = decltype(v)::value;
            if (track) stream_past ? go(step_update_kernel<V, true, true>) : go(step_update_kernel<V, true, false>);
            else stream_past ? go(step_update_kernel<V, false, true>) : go(step_update_kernel<V, false, false>);
        };
        switch (variant) {
        case PEX_ADAM: pick(std::integral_constant<int, PEX_ADAM>{}); break;
        case PEX_MICROADAM: pick(std::integral_constant<int, PEX_MICROADAM>{}); break;
        case PEX_MICROADAM_VAR: pick(std::integral_constant<int, PEX_MICROADAM_VAR>{}); break;
        case PEX_MICROADAM_MSQ: pick(std::integral_constant<int, PEX_MICROADAM_MSQ>{}); break;
        }
        if (track) step_moments_kernel<<<dim3(n), dim3(256), 0, stream>>>(g, partial, sums + 2 * at);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace pex
