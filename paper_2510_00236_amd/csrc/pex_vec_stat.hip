// pex_vec_stat.hip -- per-example statistics of vector parameters (offsets, elementwise scales).
//
// An offset added on the batch and the length axis is a contraction of the cotangents with a vector of ones
// (App. B, "Affine operations"): its per-example gradient is v_b[j] = sum_t A[b,t,j]; an elementwise scale
// applied to an activation C has v_b[j] = sum_t A[b,t,j] * C[b,t,j].  The statistic is s = sum_b phi(v_b), phi as
// for weight matrices (Sec. 2.3).  Every input byte is read once and the arithmetic is one FMA per element, so
// the bound is HBM bandwidth: B*T*d*sizeof(element) bytes per operand.
//
// Two kernels, both deterministic (fixed summation order, no atomics):
//   vec_partial_kernel   block = 64 column lanes x 4 row lanes; a lane owns VEC consecutive columns (16 bytes) and
//                        every 4th row of one range of tokens of one example; the four row lanes are summed
//                        through LDS and the block writes partial[b][range][columns] in fp32;
//   vec_finalize_kernel  per column: v_b = sum over ranges, then the requested phi, then sum over b (both dealt to the
//                        lanes of a block, combined in a fixed order).
// The partial sums are B * ranges * d floats: the per-example gradients of a *vector* parameter, which is the one
// place where holding them is cheap (B*d, not B*din*dout).
#include <type_traits>

#include "pex_internal.h"

namespace pex {
namespace {

constexpr int CW = 64, RW = 4;   // column lanes and row lanes of a block

template <typename TIn> struct VecOf;
template <> struct VecOf<uint16_t> { static constexpr int N = 8; };   // 8 bf16 = 16 bytes
template <> struct VecOf<float> { static constexpr int N = 4; };      // 4 fp32 = 16 bytes

__device__ __forceinline__ float widen(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ float widen(float f) { return f; }

template <typename TIn, int VEC>
__device__ __forceinline__ void load_vec(const TIn* p, float (&v)[VEC])
{
    if constexpr (VEC == 1) v[0] = widen(p[0]);
    else {
        typedef __attribute__((ext_vector_type(4))) unsigned int u4;
        const u4 raw = __builtin_nontemporal_load((const u4*)p);
        if constexpr (sizeof(TIn) == 2) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[2 * e] = __uint_as_float(raw[e] << 16);
                v[2 * e + 1] = __uint_as_float(raw[e] & 0xffff0000u);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(raw[e]);
        }
    }
}

// partial[(b * nrange + range) * d + j] = sum over the tokens of the range of A[b,t,j] * (HAS_C ? C[b,t,j] : 1), for the columns
// of block `colblock`; `row` = b * nrange + range
template <typename TIn, int VEC, bool HAS_C>
__device__ __forceinline__ void partial_sums(const TIn* __restrict__ A, const TIn* __restrict__ C, int T, int64_t d, int nrange, int rows_per_range,
                                             float* __restrict__ partial, int64_t colblock, int row, float (&red)[RW][CW][VEC])
{
    const int cl = threadIdx.x % CW, rl = threadIdx.x / CW;
    const int64_t j = (colblock * CW + cl) * VEC;
    const int b = row / nrange, range = row % nrange;
    const int t0 = range * rows_per_range;
    const int t1 = (t0 + rows_per_range < T) ? t0 + rows_per_range : T;
    float acc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
    if (j < d) {
        const TIn* a = A + ((int64_t)b * T) * d + j;
        const TIn* c = HAS_C ? C + ((int64_t)b * T) * d + j : nullptr;
        int t = t0 + rl;
        // four rows in flight per lane
        for (; t + 3 * RW < t1; t += 4 * RW) {
            float x[4][VEC], y[4][VEC];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                load_vec<TIn, VEC>(a + (int64_t)(t + u * RW) * d, x[u]);
                if (HAS_C) load_vec<TIn, VEC>(c + (int64_t)(t + u * RW) * d, y[u]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[e] = HAS_C ? fmaf(x[u][e], y[u][e], acc[e]) : acc[e] + x[u][e];
        }
        for (; t < t1; t += RW) {
            float x0[VEC], y0[VEC];
            load_vec<TIn, VEC>(a + (int64_t)t * d, x0);
            if (HAS_C) load_vec<TIn, VEC>(c + (int64_t)t * d, y0);
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[e] = HAS_C ? fmaf(x0[e], y0[e], acc[e]) : acc[e] + x0[e];
        }
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) red[rl][cl][e] = acc[e];
    __syncthreads();
    if (rl == 0 && j < d) {
        float* dst = partial + ((int64_t)b * nrange + range) * d + j;
#pragma unroll
        for (int e = 0; e < VEC; ++e) dst[e] = ((red[0][cl][e] + red[1][cl][e]) + red[2][cl][e]) + red[3][cl][e];
    }
}

template <typename TIn, int VEC, bool HAS_C>
__global__ __launch_bounds__(CW * RW) void vec_partial_kernel(const TIn* __restrict__ A, const TIn* __restrict__ C, int T, int64_t d,
                                                              int nrange, int rows_per_range, float* __restrict__ partial)
{
    __shared__ float red[RW][CW][VEC];
    partial_sums<TIn, VEC, HAS_C>(A, C, T, d, nrange, rows_per_range, partial, blockIdx.x, blockIdx.y, red);
}

// Second pass: per column v_b = sum over the ranges, phi, sum over the examples, the partial sums fresh in the caches.
//
// Wide blocks: 64 columns, the examples dealt to four lanes (b mod 4), each sums its phi(v_b) in ascending b with eight ranges in
// flight, the four lanes are combined in lane order.  256 contiguous bytes of a row per wave: for vectors of many columns, and
// for chains of a few loads (ceil(B / 4) * ceil(nrange / 8), about half a microsecond each).
__device__ __forceinline__ void finalize_wide(const float* __restrict__ partial, int B, int nrange, int64_t d, float* __restrict__ s_id,
                                              float* __restrict__ s_sq, float* __restrict__ s_sign, unsigned block)
{
    __shared__ float red[3][RW][CW];
    const int cl = threadIdx.x % CW, bl = threadIdx.x / CW;
    const int64_t j = (int64_t)block * CW + cl;
    float a_id = 0.f, a_sq = 0.f, a_sg = 0.f;
    if (j < d) {
        for (int b = bl; b < B; b += RW) {
            const float* p = partial + (int64_t)b * nrange * d + j;
            float v = 0.f;
            int r = 0;
            for (; r + 8 <= nrange; r += 8) {
                float x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = p[(int64_t)(r + u) * d];
#pragma unroll
                for (int u = 0; u < 8; ++u) v += x[u];
            }
            for (; r < nrange; ++r) v += p[(int64_t)r * d];
            a_id += v;
            a_sq = fmaf(v, v, a_sq);
            a_sg += (float)((v > 0.f) - (v < 0.f));
        }
    }
    red[0][bl][cl] = a_id;
    red[1][bl][cl] = a_sq;
    red[2][bl][cl] = a_sg;
    __syncthreads();
    if (bl == 0 && j < d) {
        if (s_id) s_id[j] = ((red[0][0][cl] + red[0][1][cl]) + red[0][2][cl]) + red[0][3][cl];
        if (s_sq) s_sq[j] = ((red[1][0][cl] + red[1][1][cl]) + red[1][2][cl]) + red[1][3][cl];
        if (s_sign) s_sign[j] = ((red[2][0][cl] + red[2][1][cl]) + red[2][2][cl]) + red[2][3][cl];
    }
}

__global__ __launch_bounds__(CW * RW) void vec_finalize_wide_kernel(const float* __restrict__ partial, int B, int nrange, int64_t d,
                                                               float* __restrict__ s_id, float* __restrict__ s_sq,
                                                               float* __restrict__ s_sign)
{
    finalize_wide(partial, B, nrange, d, s_id, s_sq, s_sign, blockIdx.x);
}

// Narrow blocks, for long chains over few columns: a block is 4 column lanes of VEC columns x EL example lanes x RL range lanes
// (256 in all); example b belongs to example lane b mod EL, its range r to range lane r mod RL.  Range lanes are added in
// order through LDS, then phi is applied; the example lanes' sums are added pairwise, always in the same order.  A block owns few
// columns -- d / (4 VEC) blocks -- and every lane has eight loads in flight of a chain of nrange / RL * B / EL.  VEC = 4 reads
// rows of any length 16 bytes at a time (a dwordx4 access needs no more than a float's alignment).
// Measured, the second pass alone, wide / narrow (us): B=64 in 2 ranges d=768 11.2 / 4.4, 8192 11.0 / 4.4; B=16 in 2 ranges
// d=768 4.4 / 3.8, 32768 4.0 / 5.4; B=2 d=768 2.6 / 3.9, 50256 2.6 / 6.8; B=1 in 128 ranges d=768 7.5 / 4.1; B=3000 d=768 241 / 28;
// B=2 d=4000001 28 / 810 (VEC = 1).
template <int VEC, int EL, int RL>
__device__ __forceinline__ void finalize_columns(const float* __restrict__ partial, int B, int nrange, int64_t d, float* __restrict__ s_id,
                                                 float* __restrict__ s_sq, float* __restrict__ s_sign, int64_t colblock)
{
    static_assert(4 * EL * RL == 256, "one lane per column group, example lane and range lane");
    typedef __attribute__((ext_vector_type(4))) float f4;
    typedef f4 __attribute__((aligned(4))) f4_u;
    __shared__ float red[EL * RL][4 * VEC];
    const int cl = threadIdx.x % 4, rl = (threadIdx.x / 4) % RL, el = threadIdx.x / (4 * RL);
    // first column of a column lane: the row's last chunk ends with the row (the columns it shares with its neighbour come out
    // the same twice)
    auto first_column = [&](int lane) {
        const int64_t c = (colblock * 4 + lane) * VEC;
        return c < d && c + VEC > d ? d - VEC : c;
    };
    const int64_t j = first_column(cl);
    float a_id[VEC], a_sq[VEC], a_sg[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) a_id[e] = a_sq[e] = a_sg[e] = 0.f;
    for (int b0 = 0; b0 < B; b0 += EL) {
        const int b = b0 + el;
        float v[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = 0.f;
        if (b < B && j < d) {
            const float* p = partial + (int64_t)b * nrange * d + j;
            auto load = [&](int r, float (&x)[VEC]) {
                if constexpr (VEC == 4) {
                    const f4 q = *(const f4_u*)(p + (int64_t)r * d);
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = q[e];
                } else x[0] = p[(int64_t)r * d];
            };
            int r = rl;
            for (; r + 7 * RL < nrange; r += 8 * RL) {
                float x[8][VEC];
#pragma unroll
                for (int u = 0; u < 8; ++u) load(r + u * RL, x[u]);
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) v[e] += x[u][e];
            }
            // the rest of the chain, at most seven: all in flight, those past the end as zeros
            float x[7][VEC];
#pragma unroll
            for (int u = 0; u < 7; ++u) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) x[u][e] = 0.f;
                if (r + u * RL < nrange) load(r + u * RL, x[u]);
            }
#pragma unroll
            for (int u = 0; u < 7; ++u)
#pragma unroll
                for (int e = 0; e < VEC; ++e) v[e] += x[u][e];
        }
        if constexpr (RL > 1) {
            __syncthreads();
#pragma unroll
            for (int e = 0; e < VEC; ++e) red[el * RL + rl][cl * VEC + e] = v[e];
            __syncthreads();
            if (rl == 0) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    v[e] = red[el * RL][cl * VEC + e];
#pragma unroll
                    for (int k = 1; k < RL; ++k) v[e] += red[el * RL + k][cl * VEC + e];
                }
            }
        }
        if (rl == 0 && b < B) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                a_id[e] += v[e];
                a_sq[e] = fmaf(v[e], v[e], a_sq[e]);
                a_sg[e] += (float)((v[e] > 0.f) - (v[e] < 0.f));
            }
        }
    }
    auto finish = [&](float* out, const float (&a)[VEC]) {
        __syncthreads();
        if (rl == 0) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) red[el][cl * VEC + e] = a[e];
        }
        for (int h = EL / 2; h >= 1; h >>= 1) {
            __syncthreads();
            for (int t = threadIdx.x; t < h * 4 * VEC; t += 256) red[t / (4 * VEC)][t % (4 * VEC)] += red[t / (4 * VEC) + h][t % (4 * VEC)];
        }
        __syncthreads();
        const int64_t c = first_column(threadIdx.x / VEC) + threadIdx.x % VEC;
        if (threadIdx.x < 4 * VEC && c < d) out[c] = red[0][threadIdx.x];
    };
    if (s_id) finish(s_id, a_id);
    if (s_sq) finish(s_sq, a_sq);
    if (s_sign) finish(s_sign, a_sg);
}

template <int VEC, int EL, int RL>
__global__ __launch_bounds__(256) void vec_finalize_kernel(const float* __restrict__ partial, int B, int nrange, int64_t d,
                                                           float* __restrict__ s_id, float* __restrict__ s_sq,
                                                           float* __restrict__ s_sign)
{
    finalize_columns<VEC, EL, RL>(partial, B, nrange, d, s_id, s_sq, s_sign, blockIdx.x);
}

// Several vectors of one batch in one launch of each pass: the offsets and scales of a layer are a few thousand columns each, and a
// launch costs about 4.5 us whatever it does.  The same blocks as one vector's launches, one vector after the other.
struct VecBatch {
    int count;
    unsigned first[VEC_BATCH + 1];   // first block of each vector
    const void *A[VEC_BATCH], *C[VEC_BATCH];
    float *partial[VEC_BATCH], *s_id[VEC_BATCH], *s_sq[VEC_BATCH], *s_sign[VEC_BATCH];
    int64_t d[VEC_BATCH];
    int nrange[VEC_BATCH], rows_per_range[VEC_BATCH], colblocks[VEC_BATCH], wide[VEC_BATCH];
    __device__ __forceinline__ int of_block(unsigned b) const
    {
        int k = 0;
        while (k + 1 < count && b >= first[k + 1]) ++k;
        return k;
    }
};

template <typename TIn>
__global__ __launch_bounds__(CW * RW) void vec_partial_batch_kernel(VecBatch v, int T)
{
    constexpr int V = VecOf<TIn>::N;
    __shared__ float red[RW][CW][V];
    const int k = v.of_block(blockIdx.x), local = (int)(blockIdx.x - v.first[k]), cb = local % v.colblocks[k], row = local / v.colblocks[k];
    const TIn *A = (const TIn*)v.A[k], *C = (const TIn*)v.C[k];
    auto go = [&](auto vec, auto has_c) {
        constexpr int VEC = decltype(vec)::value;
        partial_sums<TIn, VEC, decltype(has_c)::value>(A, C, T, v.d[k], v.nrange[k], v.rows_per_range[k], v.partial[k], cb, row,
                                                       reinterpret_cast<float (&)[RW][CW][VEC]>(red));
    };
    constexpr std::integral_constant<int, V> wide{};
    constexpr std::integral_constant<int, 1> one{};
    if (v.wide[k]) C ? go(wide, std::true_type{}) : go(wide, std::false_type{});
    else C ? go(one, std::true_type{}) : go(one, std::false_type{});
}

__global__ __launch_bounds__(CW * RW) void vec_finalize_wide_batch_kernel(VecBatch v, int B)
{
    const int k = v.of_block(blockIdx.x);
    finalize_wide(v.partial[k], B, v.nrange[k], v.d[k], v.s_id[k], v.s_sq[k], v.s_sign[k], blockIdx.x - v.first[k]);
}

template <int EL, int RL>
__global__ __launch_bounds__(256) void vec_finalize_batch_kernel(VecBatch v, int B)
{
    const int k = v.of_block(blockIdx.x);
    finalize_columns<4, EL, RL>(v.partial[k], B, v.nrange[k], v.d[k], v.s_id[k], v.s_sq[k], v.s_sign[k], blockIdx.x - v.first[k]);
}

// a dwordx4 load takes whole 16-byte chunks of rows here
template <typename TIn>
bool whole_chunks(const void* A, const void* C, int64_t d)
{
    return d % VecOf<TIn>::N == 0 && ((((uintptr_t)A | (uintptr_t)C) & 15u) == 0);
}

template <typename TIn>
hipError_t launch_typed(const TIn* A, const TIn* C, int64_t B, int64_t T, int64_t d, const VecPlan& plan, float* partial,
                        hipStream_t stream)
{
    constexpr int V = VecOf<TIn>::N;
    const bool wide = whole_chunks<TIn>(A, C, d);
    const int vec = wide ? V : 1;
    const dim3 grid((unsigned)((d + (int64_t)CW * vec - 1) / ((int64_t)CW * vec)), (unsigned)(B * plan.nrange));
    const dim3 block(CW * RW);
#define PEX_VEC_LAUNCH(VEC, HAS_C) \
    vec_partial_kernel<TIn, VEC, HAS_C><<<grid, block, 0, stream>>>(A, C, (int)T, d, plan.nrange, plan.rows_per_range, partial)
    if (wide) {
        if (C) PEX_VEC_LAUNCH(V, true);
        else PEX_VEC_LAUNCH(V, false);
    } else {
        if (C) PEX_VEC_LAUNCH(1, true);
        else PEX_VEC_LAUNCH(1, false);
    }
#undef PEX_VEC_LAUNCH
    return hipGetLastError();
}

}  // namespace

VecPlan plan_vec_stat(int64_t B, int64_t T, int64_t d, pex_dtype dt)
{
    // as many blocks as are resident at once (eight per compute unit) and no more, so that there is no second,
    // mostly empty round of blocks; ranges of at least 32 tokens
    VecPlan p{};
    const int vec = dt == PEX_BF16 ? 8 : 4;
    const int64_t chunks = (d + CW * vec - 1) / (CW * vec);
    int64_t nrange = 2048 / (chunks * B);
    const int64_t max_range = (T + 31) / 32;
    if (nrange > max_range) nrange = max_range;
    if (nrange < 1) nrange = 1;
    int64_t rows = (T + nrange - 1) / nrange;
    rows = (rows + RW - 1) / RW * RW;
    nrange = (T + rows - 1) / rows;
    p.nrange = (int)nrange;
    p.rows_per_range = (int)rows;
    p.ws_bytes = (size_t)B * (size_t)nrange * (size_t)d * sizeof(float);
    return p;
}

namespace {

// The narrow blocks' two-stage sum costs about three chain steps of the wide ones; beyond one block per compute unit, every 450
// blocks of sixteen columns cost another, every 300 where a step is a single load (measurements above the kernels; B=84 d=119314
// in one range, whole call: wide 72 us, narrow 84).
bool wide_second_pass(int64_t B, int64_t d, const VecPlan& plan)
{
    const int64_t narrow = (d + 15) / 16, chain = ((B + RW - 1) / RW) * ((plan.nrange + 7) / 8);
    return chain < 3 + (narrow > 256 ? (narrow - 256) / (plan.nrange == 1 ? 300 : 450) : 0);
}

// four columns a lane (short rows of odd length: more blocks; B=3000 d=77 22 against 27 us)
bool in_quads(int64_t d) { return d % 4 == 0 || d >= 512; }

hipError_t finalize_one(int64_t B, int64_t d, const VecPlan& plan, const float* partial, float* s_id, float* s_sq, float* s_sign, hipStream_t stream)
{
    if (wide_second_pass(B, d, plan)) {
        vec_finalize_wide_kernel<<<dim3((unsigned)((d + CW - 1) / CW)), dim3(CW * RW), 0, stream>>>(partial, (int)B, plan.nrange, d, s_id, s_sq, s_sign);
        return hipGetLastError();
    }
    // example lanes for the batch, the rest of the block to the ranges
    const bool quads = in_quads(d);
    const dim3 grid((unsigned)(quads ? (d + 15) / 16 : (d + 3) / 4)), block(256);
    auto go = [&](auto kern) { kern<<<grid, block, 0, stream>>>(partial, (int)B, plan.nrange, d, s_id, s_sq, s_sign); };
    if (B > 16) quads ? go(vec_finalize_kernel<4, 64, 1>) : go(vec_finalize_kernel<1, 64, 1>);
    else if (B > 4) quads ? go(vec_finalize_kernel<4, 16, 4>) : go(vec_finalize_kernel<1, 16, 4>);
    else quads ? go(vec_finalize_kernel<4, 4, 16>) : go(vec_finalize_kernel<1, 4, 16>);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_vec_stat(const void* A, const void* C, int64_t B, int64_t T, int64_t d, pex_dtype dt, const VecPlan& plan,
                           float* partial, float* s_id, float* s_sq, float* s_sign, hipStream_t stream)
{
    const hipError_t e = dt == PEX_F32 ? launch_typed((const float*)A, (const float*)C, B, T, d, plan, partial, stream)
                                       : launch_typed((const uint16_t*)A, (const uint16_t*)C, B, T, d, plan, partial, stream);
    return e != hipSuccess ? e : finalize_one(B, d, plan, partial, s_id, s_sq, s_sign, stream);
}

hipError_t launch_vec_stat_batch(const pex_vec_item* items, int count, int64_t B, int64_t T, pex_dtype dt, void* workspace, hipStream_t stream)
{
    VecBatch v{};
    char* ws = (char*)workspace;
    unsigned at = 0;
    for (int k = 0; k < count; ++k) {
        const pex_vec_item& it = items[k];
        const VecPlan plan = plan_vec_stat(B, T, it.d, dt);
        const bool wide = dt == PEX_F32 ? whole_chunks<float>(it.A, it.C, it.d) : whole_chunks<uint16_t>(it.A, it.C, it.d);
        const int64_t cols = (int64_t)CW * (wide ? (dt == PEX_F32 ? 4 : 8) : 1);
        v.first[k] = at;
        v.A[k] = it.A;
        v.C[k] = it.C;
        v.partial[k] = (float*)ws;
        v.d[k] = it.d;
        v.nrange[k] = plan.nrange;
        v.rows_per_range[k] = plan.rows_per_range;
        v.wide[k] = wide;
        v.colblocks[k] = (int)((it.d + cols - 1) / cols);
        at += (unsigned)((int64_t)v.colblocks[k] * B * plan.nrange);
        ws += vec_batch_bytes(plan);
    }
    v.count = count;
    if (dt == PEX_F32) vec_partial_batch_kernel<float><<<dim3(at), dim3(CW * RW), 0, stream>>>(v, (int)T);
    else vec_partial_batch_kernel<uint16_t><<<dim3(at), dim3(CW * RW), 0, stream>>>(v, (int)T);
    hipError_t e = hipGetLastError();
    // second pass: together what runs on wide blocks (five vectors of a block of few examples: four launches of 4.6 us less), and what runs on
    // narrow blocks of four columns a lane
    VecBatch second[2] = {};
    unsigned blocks[2] = {0, 0};
    for (int k = 0; k < count && e == hipSuccess; ++k) {
        const pex_vec_item& it = items[k];
        const VecPlan plan = plan_vec_stat(B, T, it.d, dt);
        const bool on_wide = wide_second_pass(B, it.d, plan);
        if (!on_wide && !in_quads(it.d)) {
            e = finalize_one(B, it.d, plan, v.partial[k], it.s_id, it.s_sq, it.s_sign, stream);
            continue;
        }
        VecBatch& n = second[on_wide];
        const int m = n.count++;
        n.first[m] = blocks[on_wide];
        n.partial[m] = v.partial[k];
        n.s_id[m] = it.s_id;
        n.s_sq[m] = it.s_sq;
        n.s_sign[m] = it.s_sign;
        n.d[m] = it.d;
        n.nrange[m] = plan.nrange;
        blocks[on_wide] += (unsigned)(on_wide ? (it.d + CW - 1) / CW : (it.d + 15) / 16);
    }
    if (e == hipSuccess && blocks[1] > 0) {
        vec_finalize_wide_batch_kernel<<<dim3(blocks[1]), dim3(CW * RW), 0, stream>>>(second[1], (int)B);
        e = hipGetLastError();
    }
    if (e != hipSuccess || blocks[0] == 0) return e;
    const VecBatch& n = second[0];
    if (B > 16) vec_finalize_batch_kernel<64, 1><<<dim3(blocks[0]), dim3(256), 0, stream>>>(n, (int)B);
    else if (B > 4) vec_finalize_batch_kernel<16, 4><<<dim3(blocks[0]), dim3(256), 0, stream>>>(n, (int)B);
    else vec_finalize_batch_kernel<4, 16><<<dim3(blocks[0]), dim3(256), 0, stream>>>(n, (int)B);
    return hipGetLastError();
}

}  // namespace pex
