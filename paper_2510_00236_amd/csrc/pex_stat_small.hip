// pex_stat_small.hip -- S = sum_b phi(X_b^T G_b) of layers that do not fill the chip: one launch, no exchange through memory (gfx950).
//
// The large kernels give a workgroup a block of 128 x 64 entries or more and fill the chip by splitting the batch over workgroups,
// whose partial sums a second launch adds; rows that are not whole 16-byte chunks are copied by a third.  On small layers that is
// the time: a launch costs about 4.5 us whatever it does, a block of 256 x 128 is mostly empty, and the tokens of an example
// run through one workgroup one slab after the other.  Here the eight waves of a workgroup share one tile of 64 x 64 (several
// statistics at once, where the waves divide the examples: 64 x 32) and divide its examples and tokens:
//   KW = 1: every wave takes every eighth example, its own sums, added up through LDS at the end;
//   KW = 8: every wave takes an eighth of the tokens of each example; M_b is added up through LDS at the end of the example, each
//           wave taking phi of an eighth of it.
// Bound by latency: a wave has two steps of loads in flight and nothing else to wait for -- no barrier, no LDS inside an example.
//   * Operands come straight from global memory as in pex_stat_f32.hip.  bf16: lane (q, p) = (lane / 16, lane % 16) loads four
//     features 4p .. of the eight tokens 8q .., eight bytes each at whatever address (rows of any length), and
//     sorts them by feature with 16 byte permutes: its operand of the 16x16x32 MFMA for four panels at once.  fp32: four
//     features of four tokens per group of 16, for the 16x16x4 MFMA.
//   * The last four (two) features of a width stand in for those past it: a tile owns each feature once.  Tokens past the end
//     are read from the last row there is and set to zero.
// Measured, in us, before -> now: square of 8 x 367 tokens, 64 x 128 fp32: 31.0 -> 15.2; sign, 36 x 32, 832 x 896 bf16: 33 -> 20 (182 tiles,
// no groups); square, 117 x 322, 58 x 184 bf16 (no copies of odd rows): 36 -> 20; weighted sum and norms, 56 x 1154, 64 x 48 bf16: 84 -> 34;
// plain, 1 x 9000, 20 x 31: one launch of 2 shares.  Rates stay low -- 8 x 827, 832 x 113 fp32 has 28 us for 2.4 GFLOP and 25 MB --
// because a wave waits for a step of loads (about 1 us of bf16) and there are two on a SIMD.  Of a small call the start (to the first two
// steps' loads) is 1.3 to 2.4 us and the end 1 to 2 (clock stamps inside the kernel), most of it code that runs once: so nothing is divided that the grid
// can hold, addresses are a scalar and one 32-bit offset, and a wave's sums leave as two stores.  Square, 3 x 20 tokens, 2669 x 504 bf16 10.1 -> 7.6 us;
// 17 x 24, 3712 x 369 15.8 -> 12.8; pair, 2 x 546, 1920 x 64 10.8 -> 9.5; 26 x 2428, 176 x 64 20.9 -> 19.9.
#include <type_traits>

#include "pex_f32.h"
#include "pex_internal.h"

namespace pex {
namespace {

typedef __attribute__((ext_vector_type(2))) unsigned int uint2_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;

constexpr int W = 8;                       // waves of a workgroup
constexpr int SM_T = 64;                   // rows of a tile; columns: 16 FN
constexpr int64_t SM_ROW_TILES = 65535;    // a dimension of the grid
constexpr int SM_CHUNK = 8192;             // at most so many rows of a plain contraction are folded into its sum together (1024 a wave) ...
constexpr int SM_SHORT = 4;                // ... of which a wave adds up this many steps at a time

// N 32-bit words at any element's address (one load: unaligned accesses are the rule on this target)
template <int N, int ALIGN>
__device__ __forceinline__ void load_words(const void* p, uint32_t (&v)[N])
{
    __builtin_memcpy(v, __builtin_assume_aligned(p, ALIGN), 4 * N);
}

template <typename TIn, int OUTS, int KW, int FN>
__global__ __launch_bounds__(W * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void stat_small_kernel(
    const TIn* __restrict__ X, const TIn* __restrict__ G, int rows_total, int seg_len, int din, int dout, int per_split, int64_t out_stride, float* __restrict__ out_id, float* __restrict__ out_sq, float* __restrict__ out_sg, const float* __restrict__ weight,
    float* __restrict__ norm_partial, int examples_total, float alpha, float nan_sign)
{
    constexpr bool BF16 = sizeof(TIn) == 2;
    constexpr bool PER_EXAMPLE = !(OUTS == F_PLAIN || OUTS == F_TOKEN);
    constexpr bool HAS_ID = !PER_EXAMPLE || (OUTS & (F_ID | F_IDW)) != 0, HAS_SQ = (OUTS & (F_SQ | F_POW)) != 0, HAS_SG = (OUTS & F_SG) != 0;
    constexpr int EW = W / KW, FM = 4;
    constexpr int R = BF16 ? 32 : 16, NR = BF16 ? 8 : 4;       // tokens of a step, of a lane
    constexpr int XW = BF16 ? 2 : 4, GW = BF16 ? FN / 2 : FN;  // words a lane loads of a token
    constexpr int ALIGN = (int)sizeof(TIn);
    constexpr int TILES = FM * FN, SL = KW == 1 ? TILES : FN / 2;      // 16 x 16 tiles of a wave, what it keeps of them after an example (fours of entries)
    static_assert(FM * 2 == W && (KW == 1 || KW == W), "a wave finishes two of the four rows of one feature");
    // What the waves add up goes through LDS in halves: entries 2h, 2h + 1 of every lane's four of a tile.  Wave w finishes those of h = w % 2 of
    // the tiles of row feature w / 2: of each of two rows FN columns side by side, one store (four of four bytes each took 2 us of a
    // launch of 5.4: sign, 8 x 21, 960 x 384).
    typedef __attribute__((ext_vector_type(2))) float float2_t;
    __shared__ float2_t red[2][W * TILES][64];
    const int lane = threadIdx.x & 63, q = lane >> 4, p = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), ew = wave / KW, kw = wave % KW;
    // grid = (column tiles, row tiles, groups): the start of a workgroup is a part of a small call's time, so it divides nothing
    const int split = (int)blockIdx.z, tile = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    const int i0 = (int)blockIdx.y * SM_T, j0 = (int)blockIdx.x * (16 * FN);

    // segment: one example; of a plain contraction an equal share of the rows (the last one may be shorter)
    const int first_example = PER_EXAMPLE ? split * per_split : 0;
    const int64_t row_begin = PER_EXAMPLE ? (int64_t)first_example * seg_len : (int64_t)split * per_split;
    int slen = seg_len, nex = per_split < examples_total - first_example ? per_split : examples_total - first_example, rows = 0;
    if constexpr (!PER_EXAMPLE) {
        rows = per_split < rows_total - (int)row_begin ? per_split : rows_total - (int)row_begin;
        const unsigned shares = ((unsigned)rows + SM_CHUNK - 1) / SM_CHUNK;
        slen = (int)(((unsigned)rows + shares - 1) / shares);
        nex = (int)(((unsigned)rows + (unsigned)slen - 1) / (unsigned)slen);
    }
    // this wave: tokens [t_begin, t_end) of examples ew, ew + EW, ...
    const int per = ((slen + R - 1) / R + KW - 1) / KW * R;
    const int t_begin = kw * per;
    auto t_end = [&](int ex) {
        int end = t_begin + per < slen ? t_begin + per : slen;
        if (!PER_EXAMPLE) {
            const int left = rows - ex * slen;
            if (end > left) end = left;
        }
        return end;
    };
    auto steps_of = [&](int ex) { const int n = t_end(ex) - t_begin; return n > 0 ? (n + R - 1) / R : 0; };

    // first of the features this lane loads: the last ones of the width where there are fewer
    const int cx = i0 + 4 * p + 4 <= din ? i0 + 4 * p : din - 4, cg = j0 + FN * p + FN <= dout ? j0 + FN * p : dout - FN;
    auto row_of = [&](int r) { return BF16 ? 8 * q + r : 4 * r + q; };
    // byte offsets inside a step: of this lane's first token, and from one token to the next
    const uint32_t x_row = (uint32_t)din * (uint32_t)sizeof(TIn), g_row = (uint32_t)dout * (uint32_t)sizeof(TIn);
    const uint32_t x_col = (uint32_t)cx * (uint32_t)sizeof(TIn), g_col = (uint32_t)cg * (uint32_t)sizeof(TIn);
    const uint32_t x_lane = (uint32_t)row_of(0) * x_row + x_col, g_lane = (uint32_t)row_of(0) * g_row + g_col;
    constexpr uint32_t ROWS_ON = BF16 ? 1 : 4;
    uint32_t xr[2][NR][XW], gr[2][NR][GW];
    int left[2];       // tokens of a slot's step that exist
    int ld_ex = ew, ld_t = t_begin;
    auto load = [&](auto SLOT) __attribute__((always_inline)) {
        constexpr int s = decltype(SLOT)::value;
        while (ld_ex < nex && ld_t >= t_end(ld_ex)) { ld_ex += EW; ld_t = t_begin; }
        left[s] = 0;
        if (ld_ex >= nex) return;
        const int n = __builtin_amdgcn_readfirstlane(t_end(ld_ex) - ld_t);
        left[s] = n;
        // (every lane of the wave is at the same token, which the compiler does not see: addresses in scalar registers)
        const int64_t row = row_begin + (int64_t)__builtin_amdgcn_readfirstlane(ld_ex) * slen + __builtin_amdgcn_readfirstlane(ld_t);
        const char* xb = (const char*)(X + row * din);
        const char* gb = (const char*)(G + row * dout);
        // the last token there is stands in for those past it
        const uint32_t rows_on = (uint32_t)((n < R ? n : R) - 1), x_last = rows_on * x_row + x_col, g_last = rows_on * g_row + g_col;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const uint32_t xo = x_lane + r * ROWS_ON * x_row, go = g_lane + r * ROWS_ON * g_row;
            load_words<XW, ALIGN>(xb + (xo < x_last ? xo : x_last), xr[s][r]);
            load_words<GW, ALIGN>(gb + (go < g_last ? go : g_last), gr[s][r]);
        }
        ld_t += R;
    };
    float4_t acc[FM][FN];
    auto clear = [&]() {
#pragma unroll
        for (int m = 0; m < FM; ++m)
#pragma unroll
            for (int n = 0; n < FN; ++n) acc[m][n] = float4_t{0.f, 0.f, 0.f, 0.f};
    };
    auto multiply = [&](auto SLOT) __attribute__((always_inline)) {
        constexpr int s = decltype(SLOT)::value;
        if (left[s] < R) {
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const bool in = row_of(r) < left[s];
#pragma unroll
                for (int w = 0; w < XW; ++w) xr[s][r][w] = in ? xr[s][r][w] : 0u;
#pragma unroll
                for (int w = 0; w < GW; ++w) gr[s][r][w] = in ? gr[s][r][w] : 0u;
            }
        }
        if constexpr (BF16) {
            // tokens 2k, 2k+1 of feature e: the halves of words e / 2
            auto operand = [&](const auto& raw, int e) {
                uint4_t f;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    f[k] = __builtin_amdgcn_perm(raw[2 * k + 1][e / 2], raw[2 * k][e / 2], e % 2 ? 0x07060302u : 0x05040100u);
                return __builtin_bit_cast(bf16x8_t, f);
            };
            bf16x8_t g[FN];
#pragma unroll
            for (int n = 0; n < FN; ++n) g[n] = operand(gr[s], n);
#pragma unroll
            for (int m = 0; m < FM; ++m) {
                const bf16x8_t x = operand(xr[s], m);
#pragma unroll
                for (int nn = 0; nn < FN; ++nn) {
                    const int n = m & 1 ? FN - 1 - nn : nn;
                    acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, g[n], acc[m][n], 0, 0, 0);
                }
            }
        } else {
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                float a[FM], b[FN];
#pragma unroll
                for (int m = 0; m < FM; ++m) a[m] = __uint_as_float(xr[s][r][m]);
#pragma unroll
                for (int n = 0; n < FN; ++n) b[n] = __uint_as_float(gr[s][r][n]);
                if (OUTS == F_TOKEN) {       // exact fp32 squares
#pragma unroll
                    for (int m = 0; m < FM; ++m) a[m] *= a[m];
#pragma unroll
                    for (int n = 0; n < FN; ++n) b[n] *= b[n];
                }
#pragma unroll
                for (int m = 0; m < FM; ++m)
#pragma unroll
                    for (int nn = 0; nn < FN; ++nn) {
                        const int n = m & 1 ? FN - 1 - nn : nn;
                        acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m], b[n], acc[m][n], 0, 0, 0);
                    }
            }
        }
    };

    // 16 x 16 tile t = m FN + n: entry r of a lane is feature `m` of the four of row lane 4q + r, feature n of column lane p
    auto row_feature = [&](int m, int r, bool& own) {
        const int c = i0 + 4 * (4 * q + r), f = (c + 4 <= din ? c : din - 4) + m;
        own = f >= c && c < din;
        return f;
    };
    auto col_feature = [&](int n, bool& own) {
        const int c = j0 + FN * p;
        own = cg + n >= c && c < dout;
    };
    // (KW = W: entry 2 (n % 2) + i of four n / 2 is row i of this wave's two, column n)
    const int mine_m = wave / 2, mine_h = wave % 2;
    auto share = [&](int w, int t, const float4_t& v) __attribute__((always_inline)) {
        red[0][w * TILES + t][lane] = float2_t{v[0], v[1]};
        red[1][w * TILES + t][lane] = float2_t{v[2], v[3]};
    };
    float4_t s_id[HAS_ID ? SL : 1], s_sq[HAS_SQ ? SL : 1], s_sg[HAS_SG ? SL : 1];
#pragma unroll
    for (int t = 0; t < SL; ++t) {
        if (HAS_ID) s_id[t] = float4_t{0.f, 0.f, 0.f, 0.f};
        if (HAS_SQ) s_sq[t] = float4_t{0.f, 0.f, 0.f, 0.f};
        if (HAS_SG) s_sg[t] = float4_t{0.f, 0.f, 0.f, 0.f};
    }
    // a plain contraction of this wave, short chains of additions at a time
    static_assert(PER_EXAMPLE || KW == W, "a plain contraction is divided by tokens");
    [[maybe_unused]] float4_t run[PER_EXAMPLE ? 1 : TILES];
    if (!PER_EXAMPLE)
#pragma unroll
        for (int t = 0; t < TILES; ++t) run[t] = float4_t{0.f, 0.f, 0.f, 0.f};
    auto shorten = [&]() {
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            run[t] += acc[t / FN][t % FN];
            acc[t / FN][t % FN] = float4_t{0.f, 0.f, 0.f, 0.f};
        }
    };
    // end of example `ex` of the group (>= nex: none, for the barriers only)
    auto fold = [&](int ex) __attribute__((always_inline)) {
        if constexpr (KW > 1) {
#pragma unroll
            for (int t = 0; t < TILES; ++t) {
                float4_t v = acc[t / FN][t % FN];
                if (!PER_EXAMPLE) {
                    v += run[t];
                    run[t] = float4_t{0.f, 0.f, 0.f, 0.f};
                }
                share(wave, t, v);
            }
            __syncthreads();
        }
        const int example = first_example + ex;
        const float w = (OUTS & F_IDW) && ex < nex ? weight[example] : 1.f;
        float part[4] = {0.f, 0.f, 0.f, 0.f};        // of a norm: four short chains of additions
        if (ex < nex) {
#pragma unroll
            for (int t = 0; t < SL; ++t) {
                float4_t v;
                if constexpr (KW == 1) v = acc[t / FN][t % FN];
                else {
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        const int tt = mine_m * FN + 2 * t + half;
                        float2_t u = red[mine_h][tt][lane];
#pragma unroll
                        for (int k = 1; k < KW; ++k) u += red[mine_h][k * TILES + tt][lane];
                        v[2 * half] = u[0];
                        v[2 * half + 1] = u[1];
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float x = v[r];
                    if (!PER_EXAMPLE || (OUTS & F_ID)) s_id[t][r] += x;
                    if (OUTS & F_IDW) s_id[t][r] = fmaf(w, x, s_id[t][r]);
                    if (OUTS & F_SQ) s_sq[t][r] = fmaf(x, x, s_sq[t][r]);
                    if (OUTS & F_POW) s_sq[t][r] += power_of(x, alpha);
                    if (OUTS & F_SG) {      // the median takes every non-zero value scaled by 2^200 to +-1, and NaN to -1
                        const float sg = __builtin_amdgcn_fmed3f(__builtin_ldexpf(x, 200), -1.0f, 1.0f);
                        s_sg[t][r] += x != x ? nan_sign : sg;
                    }
                    if (OUTS & F_NORM) {
                        bool mine_i, mine_j;
                        row_feature(KW == 1 ? t / FN : mine_m, KW == 1 ? r : 2 * mine_h + r % 2, mine_i);
                        col_feature(KW == 1 ? t % FN : 2 * t + r / 2, mine_j);
                        const float u = mine_i && mine_j ? x : 0.f;      // (on both factors: an infinity that is not ours times zero is NaN)
                        part[r] = fmaf(u, u, part[r]);
                    }
                }
            }
            if (OUTS & F_NORM) {
                float norm = (part[0] + part[1]) + (part[2] + part[3]);
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) norm += __shfl_xor(norm, off);
                if (lane == 0) norm_partial[((int64_t)tile * KW + kw) * examples_total + example] = norm;
            }
        }
        if constexpr (KW > 1) __syncthreads();
        clear();
    };

    constexpr std::integral_constant<int, 0> S0{};
    constexpr std::integral_constant<int, 1> S1{};
    clear();
    load(S0);
    load(S1);
    const int rounds = (nex + EW - 1) / EW;       // folds, the same number in every wave
    int round = 0, done = 0, need = ew < nex ? steps_of(ew) : 0;
    auto settle = [&]() __attribute__((always_inline)) {                          // fold what is complete, examples without a step of this wave's included
        while (round < rounds && done >= need) {
            fold(ew + round * EW);
            ++round;
            done = 0;
            need = ew + round * EW < nex ? steps_of(ew + round * EW) : 0;
        }
    };
    if (need == 0) settle();
    auto step = [&](auto SLOT) __attribute__((always_inline)) {
        multiply(SLOT);
        load(SLOT);
        ++done;
        if (!PER_EXAMPLE && done % SM_SHORT == 0) shorten();
        settle();
    };
    while (left[0] > 0) {
        step(S0);
        if (left[1] <= 0) break;
        step(S1);
    }
    if (OUTS & F_NORM) return;

    // the groups' sums, each wave an eighth of the tile.  (The last columns of a width may be another lane's or tile's too, who stores the same.)
    auto finish = [&](const float4_t* sums, float* __restrict__ out, bool first) __attribute__((always_inline)) {
        float v[2][FN];
        if constexpr (EW > 1) {
            if (!first) __syncthreads();
#pragma unroll
            for (int t = 0; t < TILES; ++t) share(wave, t, sums[t]);
            __syncthreads();
        }
#pragma unroll
        for (int n = 0; n < FN; ++n) {
            if constexpr (EW == 1) {
                v[0][n] = sums[n / 2][2 * (n % 2)];
                v[1][n] = sums[n / 2][2 * (n % 2) + 1];
            } else {
                const int t = mine_m * FN + n;
                float2_t u = red[mine_h][t][lane];
#pragma unroll
                for (int e = 1; e < EW; ++e) u += red[mine_h][e * TILES + t][lane];
                v[0][n] = u[0];
                v[1][n] = u[1];
            }
        }
        typedef __attribute__((ext_vector_type(FN))) float row_t;
        typedef row_t __attribute__((aligned(4))) row_u;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            bool mine_i;
            const int i = row_feature(mine_m, 2 * mine_h + r, mine_i);
            row_t x;
#pragma unroll
            for (int n = 0; n < FN; ++n) x[n] = v[r][n];
            if (mine_i && j0 + FN * p < dout) *(row_u*)(out + (int64_t)split * out_stride + (int64_t)i * dout + cg) = x;
        }
    };
    if constexpr (HAS_ID) finish(s_id, out_id, true);
    if constexpr (HAS_SQ) finish(s_sq, out_sq, !HAS_ID);
    if constexpr (HAS_SG) finish(s_sg, out_sg, !HAS_ID && !HAS_SQ);
}

template <typename TIn, int OUTS, int KW, int FN>
hipError_t launch_small(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, const StatPlan& plan, float* out_id, float* out_sq,
                        float* out_sg, hipStream_t stream, const float* weight, float* norm_partial, float alpha, float nan_sign)
{
    const int64_t tiles_n = (dout + 16 * FN - 1) / (16 * FN), tiles_m = (din + SM_T - 1) / SM_T;
    if (tiles_m > SM_ROW_TILES || plan.nsplit > 65535) return hipErrorInvalidValue;       // (small_supports asks for the first; plans have at most 1024 groups)
    stat_small_kernel<TIn, OUTS, KW, FN><<<dim3((unsigned)tiles_n, (unsigned)tiles_m, (unsigned)plan.nsplit), dim3(W * 64), 0, stream>>>(
        (const TIn*)X, (const TIn*)G, (int)(B * T), (int)T, (int)din, (int)dout, (int)plan.per_split, din * dout, out_id, out_sq, out_sg, weight, norm_partial, (int)B, alpha, nan_sign);
    return hipGetLastError();
}

template <typename TIn>
hipError_t launch_typed(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, Mode mode, const StatPlan& plan, float* out,
                        hipStream_t stream, const float* weight, float* norm_partial, float alpha, float nan_sign)
{
    auto go = [&](auto outs, float* id, float* sq, float* sg) {
        constexpr int O = decltype(outs)::value;
        return plan.small_kw == 1 ? launch_small<TIn, O, 1, 4>(X, G, B, T, din, dout, plan, id, sq, sg, stream, weight, norm_partial, alpha, nan_sign)
                                  : launch_small<TIn, O, 8, 4>(X, G, B, T, din, dout, plan, id, sq, sg, stream, weight, norm_partial, alpha, nan_sign);
    };
    switch (mode) {
    case MODE_IDENTITY: return launch_small<TIn, F_PLAIN, 8, 4>(X, G, B, T, din, dout, plan, out, nullptr, nullptr, stream, nullptr, nullptr, 0.f, 0.f);
    case MODE_SQUARE: return go(std::integral_constant<int, F_SQ>{}, nullptr, out, nullptr);
    case MODE_SIGN: return go(std::integral_constant<int, F_SG>{}, nullptr, nullptr, out);
    case MODE_WEIGHTED: return go(std::integral_constant<int, F_IDW>{}, out, nullptr, nullptr);
    case MODE_POWER: return go(std::integral_constant<int, F_POW>{}, nullptr, out, nullptr);
    case MODE_NORMS: return go(std::integral_constant<int, F_NORM>{}, nullptr, nullptr, nullptr);
    case MODE_TOKEN_SQ:
        if constexpr (sizeof(TIn) == 4)
            return launch_small<TIn, F_TOKEN, 8, 4>(X, G, B, T, din, dout, plan, out, nullptr, nullptr, stream, nullptr, nullptr, 0.f, 0.f);
    }
    return hipErrorInvalidValue;
}

// NaN counts as -1 on bf16 layers of whole 16-byte chunks, as 0 on all others
float sign_of_nan(int64_t din, int64_t dout, pex_dtype dt) { return dt == PEX_BF16 && din % 8 == 0 && dout % 8 == 0 ? -1.f : 0.f; }

}  // namespace

bool small_supports(int64_t T, int64_t din, int64_t dout, pex_dtype dt, Mode mode)
{
    // a lane reads four features of a row; 32-bit byte offsets inside a step; the tokens of an example are counted in 32 bits
    if (din < 4 || dout < 4 || din > ((int64_t)1 << 24) || dout > ((int64_t)1 << 24) || T > ((int64_t)1 << 30)) return false;
    if (dt == PEX_BF16 && mode == MODE_TOKEN_SQ) return false;
    // row tiles are a grid dimension of at most 65535
    return small_tiles(din, dout) < ((int64_t)1 << 22) && (din + SM_T - 1) / SM_T <= SM_ROW_TILES;
}

int64_t small_tiles(int64_t din, int64_t dout, bool half) { return ((din + SM_T - 1) / SM_T) * (half ? (dout + 31) / 32 : (dout + SM_T - 1) / SM_T); }

hipError_t launch_stat_small(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt, Mode mode, const StatPlan& plan,
                             float* out, hipStream_t stream, const float* weight, float* norm_partial, float alpha)
{
    const float nan_sign = sign_of_nan(din, dout, dt);
    return dt == PEX_F32 ? launch_typed<float>(X, G, B, T, din, dout, mode, plan, out, stream, weight, norm_partial, alpha, nan_sign)
                         : launch_typed<uint16_t>(X, G, B, T, din, dout, mode, plan, out, stream, weight, norm_partial, alpha, nan_sign);
}

hipError_t launch_stat_small_multi(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt, const StatPlan& plan,
                                   float* out_id, float* out_sq, float* out_sg, hipStream_t stream)
{
    const float nan_sign = sign_of_nan(din, dout, dt);
    auto go = [&](auto outs) {
        constexpr int O = decltype(outs)::value;
        auto typed = [&](auto zero) {
            typedef decltype(zero) TIn;
            return plan.small_kw == 8 ? launch_small<TIn, O, 8, 4>(X, G, B, T, din, dout, plan, out_id, out_sq, out_sg, stream, nullptr, nullptr, 0.f, nan_sign)
                                      : launch_small<TIn, O, 1, 2>(X, G, B, T, din, dout, plan, out_id, out_sq, out_sg, stream, nullptr, nullptr, 0.f, nan_sign);
        };
        return dt == PEX_F32 ? typed(0.f) : typed((uint16_t)0);
    };
    if (out_id && out_sq && out_sg) return go(std::integral_constant<int, F_ID | F_SQ | F_SG>{});
    if (out_id && out_sq) return go(std::integral_constant<int, F_ID | F_SQ>{});
    if (out_id && out_sg) return go(std::integral_constant<int, F_ID | F_SG>{});
    if (out_sq && out_sg) return go(std::integral_constant<int, F_SQ | F_SG>{});
    return hipErrorInvalidValue;
}

}  // namespace pex
