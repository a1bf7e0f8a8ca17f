// pex_stat_f32_split.hip -- fp32 layers on the bf16 matrix cores: every operand as the sum of three bf16 pieces (gfx950).
//
// An fp32 value has 24 significant bits, a bf16 value 8: x = x1 + x2 + x3 with x1 = bf16(x), x2 = bf16(x - x1),
// x3 = bf16(x - x1 - x2), each rounded to nearest, and all three differences exact (see "range" below).  Of the nine products of
// pieces x2 g3, x3 g2 and x3 g3 are left out: together at most 2^-24 of x g, half a unit in the last place of an fp32 product,
// 2^-27 as a root mean square.  The other six are exact in fp32 and run through v_mfma_f32_16x16x32_bf16.
// Sums: that instruction rounds what it adds to its third operand worse than to nearest (with one token and the products added to
// M_b one after the other the error was 5.4e-8 of the 2-norm, 2.5e-8 by fp32 products), so nothing is added to M_b by it.  Of
// every 32 tokens the five small products (at most 2^-8 of the large one) are one chain, x1 g1 another, both from zero; the sum
// of the two is added to M_b by vector instructions.  Against 64-bit sums, by fp32 products (pex_stat_f32.hip) and here, in 1e-8 of the
// 2-norm (B=8, T=1024, 1152x1280): identity 57.6, 11.8, square 55.8, 11.7; X without its negative values 40.7, 11.6 and 39.5,
// 11.5; all values 1.0039, where the products left out are largest, 5.8 and 0.02.  Examples of one non-zero token 2.5, 2.6; of two
// that are not among the same 32 3.0, 3.7; four 4.1, 4.2; sixteen 6.1, 6.2, next to each other 7.3, 3.1.
//
// Bound: the bf16 MFMA pipe at six products, 16 / 6 of the fp32 pipe's rate, and the vector instructions beside it.  Measured,
// B=8, T=1024, 2048x4096: phi = square 0.69 ms = 200 TFLOP/s (pex_stat_f32.hip: 0.95 ms, 145; all products added to M_b by the
// MFMA 0.60).
//   * A workgroup of four waves owns a 128 x 128 block, a wave 64 x 64 of it; two workgroups share a compute unit, and while
//     one of them splits its next 32 tokens the other one multiplies.
//   * Splitting takes 6.5 vector instructions per value; each value is split once per workgroup and the pieces are shared through
//     LDS (48 KB).  A wave that split its own fragments would do the work twice.
//   * A thread loads 4 features of 8 tokens with 16-byte loads (16 lanes read 256 contiguous bytes of a token), one slab ahead of
//     the one being multiplied, and writes 12 pieces of 8 tokens, each the operand of one MFMA lane.  The position of a
//     piece inside the 256 bytes of its panel and tokens is permuted so that both the eight lanes of a write and the eight
//     lanes of a read fall into different banks.
//   * The products of one 16 x 16 tile follow each other (side by side with three neighbours they took 0.70 ms), the sums of a tile
//     go to M_b under the products of the next.  Two of each chain, M_b, the sum, the fragments and the loads in flight fill the 256
//     registers: lane numbers and offsets are formed where they are used.
//   * Blocks overlap at the edge of a width as the tiles of pex_stat_f32.hip do; rows past the end of an example lie outside
//     the buffer descriptor and arrive as zeros.
//   * Identity and square from one contraction: the registers of two waves per SIMD hold M_b and one sum.  S_id is added up in
//     memory (the first example of a group stores, the L2 adds the others; every entry belongs to one lane, which adds in
//     ascending order), with nothing waiting for it.
//
// Range: both operands are scaled by 2^24 before they are split, so that the last piece of the smallest fp32 value is a normal
// bf16, and M_b by 2^-48 where it leaves the accumulators.  Values from 2^104 and results from 2^80 on become infinite: a
// wave whose results are not finite makes its tile again with the fp32 MFMA from the operands as they are, same results as
// pex_stat_f32.hip (also where a square does overflow, where that changes nothing).  All tiles again: 1.55 ms at the shape above.
#include <type_traits>

#include "pex_f32.h"
#include "pex_internal.h"
#include "pex_lds_dma.h"
#include "pex_tile_map.h"

namespace pex {
namespace {

typedef __attribute__((ext_vector_type(2))) float float2_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;

constexpr int S_T = 128, S_ROWS = 32, S_THREADS = 256;
constexpr int S_PANELS = 2 * S_T / 16;                 // panels of 16 features: X's, then G's
constexpr int S_PIECE = S_PANELS * 64;                 // 16-byte units of one piece of a slab
constexpr float S_SCALE = 0x1p24f, S_UNSCALE = 0x1p-48f;      // of an operand, of M_b

// The pieces of two values (tokens t, t+1 of a feature), two bf16 to a dword
__device__ __forceinline__ void split_pair(float a, float b, uint32_t (&piece)[3])
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const uint32_t u = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2_t{a, b}), bf16x2_t));
        piece[k] = u;
        a -= __uint_as_float(u << 16);
        b -= __uint_as_float(u & 0xffff0000u);
    }
}

// This lane's number, formed where it is asked for: a register less beside the main loop
__device__ __forceinline__ int fresh_lane()
{
    uint32_t zero = 0;
    asm volatile("" : "+s"(zero));
    return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
}

template <int OUTS>
__global__ __launch_bounds__(S_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void stat_f32_split_kernel(
    const float* __restrict__ X, const float* __restrict__ G, int64_t rows_total, int seg_len, int din, int dout, int64_t rows_per_split,
    int window_rows, int blocks_m, int blocks_n, int64_t out_stride, float* __restrict__ out_id, float* __restrict__ out_sq,
    const float* __restrict__ weight, float* __restrict__ norm_partial, int examples_total, float alpha)
{
    constexpr bool PER_EXAMPLE = !(OUTS == F_PLAIN || OUTS == F_TOKEN);
    constexpr bool ID_IN_MEMORY = (OUTS & F_ID) != 0;
    constexpr bool HAS_SUM = (OUTS & F_NORM) == 0;      // a second register tile: the one statistic (of two: the square)
    __shared__ uint4_t pieces[3 * S_PIECE];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int split, bm, bn;
    map_workgroup(blocks_m, blocks_n, split, bm, bn);
    const int own_i = bm * S_T, own_j = bn * S_T;       // first entry that is this block's own
    const int i0 = own_i + S_T <= din ? own_i : (din > S_T ? din - S_T : 0);
    const int j0 = own_j + S_T <= dout ? own_j : (dout > S_T ? dout - S_T : 0);

    const int64_t row_begin = (int64_t)split * rows_per_split;
    int64_t row_end = row_begin + rows_per_split;
    if (row_end > rows_total) row_end = rows_total;
    const int64_t rows = row_end - row_begin;
    // segment: one example; a plain contraction is folded into its sum every F_CHUNK rows (shorter chains of additions)
    const int slen = PER_EXAMPLE ? seg_len : F_CHUNK;
    const int nst = (slen + S_ROWS - 1) / S_ROWS;
    const int64_t total = PER_EXAMPLE ? rows / seg_len * nst : (rows + S_ROWS - 1) / S_ROWS;

    // ---- loader: waves 0 and 1 take X, waves 2 and 3 G; lane (o, l) = (lane / 32, lane % 32) of a wave tokens 8q .. 8q+7 of
    // the slab with q = 2 * (wave % 2) + o, features 4l .. 4l+3 of the block (whole chunks: a width below a block's is a multiple of 4)
    const int side = wave >> 1, oct = (wave & 1) * 2 + (lane >> 5), ll = lane & 31;
    const int width = side ? dout : din, c0 = side ? j0 : i0;
    const uint32_t voff = c0 + 4 * ll < width ? (uint32_t)(8 * oct * width + c0 + 4 * ll) * 4u : F_OUTSIDE;
    const uint32_t pitch = (uint32_t)width * 4u;
    // windows as in pex_stat_f32.hip: runs of rows of one segment that one descriptor covers
    const float* base = (side ? G : X) + row_begin * width;
    const int win_rows = window_rows < slen ? window_rows : slen;      // a multiple of S_ROWS, or the whole segment
    int64_t rows_left = rows;
    int seg_left = slen, win_slabs = 0;
    uint32_t at = 0;
    __amdgpu_buffer_rsrc_t rs;
    auto next_window = [&]() {
        int n = win_rows < seg_left ? win_rows : seg_left;
        if (n > rows_left) n = (int)rows_left;
        rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, n * width * 4, 0x00020000);
        at = 0;
        base += (int64_t)n * width;
        rows_left -= n;
        seg_left -= n;
        if (seg_left <= 0) seg_left = slen;
        win_slabs = n > 0 ? (n + S_ROWS - 1) / S_ROWS : 1 << 30;
    };
    uint4_t raw[8];
    auto load = [&]() {
#pragma unroll
        for (int r = 0; r < 8; ++r) raw[r] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(voff + at + (uint32_t)r * pitch), 0, 0);
        at += pitch * S_ROWS;
        if (--win_slabs == 0) next_window();
    };
    // Position of slot s (feature s of a panel) inside the 16 units of panel a and tokens q, by bits: s2 + 2 (s3^s1) + 4 (a0^s0) + 8 s1.
    // A write (lanes: s3, s2 and panels) and a read (lanes: s2, s1, s0) of eight lanes both cover eight different units mod 8.
    auto put = [&]() {
        const int fl = fresh_lane(), wpos = (side * 8 + ((fl & 31) >> 2)) * 64 + ((wave & 1) * 2 + (fl >> 5)) * 16 + (fl & 7);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint4_t u[3];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float a = __uint_as_float(raw[2 * q][e]), b = __uint_as_float(raw[2 * q + 1][e]);
                if (OUTS == F_TOKEN) { a *= a; b *= b; }     // exact fp32 squares
                a *= S_SCALE;
                b *= S_SCALE;
                uint32_t piece[3];
                split_pair(a, b, piece);
#pragma unroll
                for (int k = 0; k < 3; ++k) u[k][q] = piece[k];
            }
            const int pos = (wpos ^ (2 * (e >> 1)) ^ (4 * (e & 1))) + 8 * (e >> 1);
#pragma unroll
            for (int k = 0; k < 3; ++k) pieces[pos + k * S_PIECE] = u[k];
        }
    };

    // ---- multiplier
    const int wm = wave >> 1, wn = wave & 1, p = lane & 15, k4 = lane >> 4;
    const int rpos = k4 * 16 + ((p >> 2) & 1) + 2 * (((p >> 3) ^ (p >> 1)) & 1) + 4 * (p & 1) + 8 * ((p >> 1) & 1);
    const int rx = wm * 256 + rpos, rg = S_PIECE / 2 + wn * 256 + rpos;
    float4_t acc[4][4], sum[HAS_SUM ? 4 : 1][4];
    auto clear = [&]() {
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                acc[m][n] = float4_t{0.f, 0.f, 0.f, 0.f};
                if (HAS_SUM) sum[m][n] = acc[m][n];
            }
    };
    auto multiply = [&]() {
        bf16x8_t g[4][3], x[2][2], x3;
        auto unit_x = [&](int m, int k) { return __builtin_bit_cast(bf16x8_t, pieces[(rx ^ (4 * (m & 1))) + m * 64 + k * S_PIECE]); };
        auto read_g = [&](int n, int k) { g[n][k] = __builtin_bit_cast(bf16x8_t, pieces[(rg ^ (4 * (n & 1))) + n * 64 + k * S_PIECE]); };
        x[0][1] = unit_x(0, 1);
        read_g(0, 1);
        read_g(0, 0);
        x3 = unit_x(0, 2);
        x[0][0] = unit_x(0, 0);
        read_g(0, 2);
#pragma unroll
        for (int n = 1; n < 4; ++n)
#pragma unroll
            for (int k = 0; k < 3; ++k) read_g(n, k);
        const float4_t zero = {0.f, 0.f, 0.f, 0.f};
        float4_t d[2], e[2];
        auto settle = [&](int t) { acc[t >> 2][t & 3] += d[t & 1] + e[t & 1]; };
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            if (m < 3) {
                x[(m + 1) & 1][1] = unit_x(m + 1, 1);
                x[(m + 1) & 1][0] = unit_x(m + 1, 0);
            }
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                const int t = 4 * m + n;
                float4_t& c = d[t & 1];
                auto add = [&](const bf16x8_t& a, int k, const float4_t& from) { c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, g[n][k], from, 0, 0, 0); };
                if (n == 0) {
                    add(x[m & 1][1], 1, zero);
                    add(x[m & 1][1], 0, c);
                    add(x3, 0, c);
                } else {
                    add(x3, 0, zero);
                    if (n == 3 && m < 3) x3 = unit_x(m + 1, 2);
                    add(x[m & 1][1], 1, c);
                    add(x[m & 1][1], 0, c);
                }
                add(x[m & 1][0], 2, c);
                e[t & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[m & 1][0], g[n][0], zero, 0, 0, 0);
                add(x[m & 1][0], 1, c);
                __builtin_amdgcn_sched_barrier(0);
                if (t > 0) settle(t - 1);
            }
        }
        settle(15);
    };

    // ---- end of an example.  Row of (m, r): ib + 16m + r; column of n: jb + 16n
    const int example0 = (int)(row_begin / seg_len);
    int example = example0;
    float check = 0.f;              // NaN once something is not finite
    float unscale = S_UNSCALE;
    // S_id in memory: byte offsets from the block's first own row; what is not this block's own gets an offset outside (rows above
    // wrap around, rows below lie past the end)
    [[maybe_unused]] int4_t mem_rsrc;
    if constexpr (ID_IN_MEMORY) {
        const int own_rows = din - own_i < S_T ? din - own_i : S_T;
        mem_rsrc = make_rsrc(out_id + (int64_t)split * out_stride + (int64_t)own_i * dout, (uint32_t)(own_rows * dout) * 4u);
    }
    auto fold = [&]() {
        const int fl = fresh_lane(), ib = i0 + wm * F_T + 4 * (fl >> 4), jb = j0 + wn * F_T + (fl & 15);
        float w = 1.f, norm = 0.f;
        if (OUTS & F_IDW) w = weight[example];
        // a norm counts what is this block's own: not its neighbour's part of an overlapping block, nothing beyond a narrow panel
        const bool whole = own_i + S_T <= din && own_j + S_T <= dout;
        if constexpr (ID_IN_MEMORY) {
            uint32_t mem_off[4];
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                const int j = jb + 16 * n;
                mem_off[n] = j >= own_j && j < dout ? (uint32_t)((ib - own_i) * dout + j) * 4u : F_OUTSIDE;
            }
            auto emit = [&](auto FIRST) {
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int n = 0; n < 4; ++n) {
                            const uint32_t row_off = (uint32_t)(16 * m + r) * (uint32_t)dout * 4u;
                            if constexpr (decltype(FIRST)::value) mem_store_f32(acc[m][n][r] * unscale, mem_off[n], row_off, mem_rsrc);
                            else mem_add_f32(acc[m][n][r] * unscale, mem_off[n], row_off, mem_rsrc);
                        }
            };
            if (example == example0) emit(std::true_type{});
            else emit(std::false_type{});
        }
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int n = 0; n < 4; ++n) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float v = acc[m][n][r] * unscale;
                    if (!PER_EXAMPLE) sum[m][n][r] += v;
                    if (OUTS & F_IDW) sum[m][n][r] = fmaf(w, v, sum[m][n][r]);
                    if (OUTS & F_SQ) sum[m][n][r] = fmaf(v, v, sum[m][n][r]);
                    if (OUTS & F_POW) sum[m][n][r] += power_of(v, alpha);
                    if (OUTS & F_SG) { sum[m][n][r] += sign_of(v); check = fmaf(v, 0.f, check); }
                    if (OUTS & F_NORM) {
                        const int i = ib + 16 * m + r, j = jb + 16 * n;
                        const bool mine = whole || (i >= own_i && i < din && j >= own_j && j < dout);
                        const float u = mine ? v : 0.f;
                        norm = fmaf(u, u, norm);
                    }
                }
                acc[m][n] = float4_t{0.f, 0.f, 0.f, 0.f};
            }
        if (OUTS & F_NORM) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) norm += __shfl_xor(norm, off);
            if (fl == 0) norm_partial[((int64_t)(bm * blocks_n + bn) * 4 + wave) * examples_total + example] = norm;
            check = fmaf(norm, 0.f, check);
        }
        ++example;
    };

    clear();
    next_window();
    load();
    int st_in_seg = 0;
    for (int64_t s = 0; s < total; ++s) {
        put();
        load();
        const bool last = ++st_in_seg == nst;
        wait_lds_and_barrier();         // the slab is written
        __builtin_amdgcn_s_setprio(1);
        multiply();
        __builtin_amdgcn_s_setprio(0);
        if (last) { st_in_seg = 0; fold(); }
        wait_lds_and_barrier();         // and read
    }
    if (!PER_EXAMPLE && st_in_seg > 0) fold();
    if (HAS_SUM && !(OUTS & F_SG)) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int n = 0; n < 4; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r) check = fmaf(sum[m][n][r], 0.f, check);
    }
    if (__any(!(check == 0.f))) {
        // once more with true fp32 products: operand lane (k4, p) is token k4 of a group of four, feature 16m + p; four groups ahead
        if (ID_IN_MEMORY) wait_vmcnt<0>();
        clear();
        example = example0;
        unscale = 1.f;
        const int fl = fresh_lane(), fp = fl & 15, fk = fl >> 4;
        for (int64_t t0 = row_begin; t0 < row_end; t0 += slen) {
            const int64_t end = t0 + slen < row_end ? t0 + slen : row_end;
            float a[2][4][4], b[2][4][4];
            // (columns past a narrow width read the next row; they are no entry's)
            auto fetch = [&](int64_t t, float (&x)[4][4], float (&g)[4][4]) {
                const int n = end - t < 16 ? (end > t ? (int)(end - t) : 0) : 16;
                const __amdgpu_buffer_rsrc_t rx2 = __builtin_amdgcn_make_buffer_rsrc((void*)(X + t * din), 0, n * din * 4, 0x00020000);
                const __amdgpu_buffer_rsrc_t rg2 = __builtin_amdgcn_make_buffer_rsrc((void*)(G + t * dout), 0, n * dout * 4, 0x00020000);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int at_x = ((4 * u + fk) * din + i0 + wm * F_T + fp) * 4, at_g = ((4 * u + fk) * dout + j0 + wn * F_T + fp) * 4;
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        x[u][m] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rx2, at_x + 64 * m, 0, 0));
                        g[u][m] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rg2, at_g + 64 * m, 0, 0));
                    }
                }
            };
            auto products = [&](float (&x)[4][4], float (&g)[4][4]) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (OUTS == F_TOKEN) {
#pragma unroll
                        for (int m = 0; m < 4; ++m) { x[u][m] *= x[u][m]; g[u][m] *= g[u][m]; }
                    }
#pragma unroll
                    for (int m = 0; m < 4; ++m)
#pragma unroll
                        for (int n = 0; n < 4; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][m], g[u][n], acc[m][n], 0, 0, 0);
                }
            };
            fetch(t0, a[0], b[0]);
            for (int64_t t = t0; t < end; t += 32) {
                fetch(t + 16, a[1], b[1]);
                products(a[0], b[0]);
                fetch(t + 32, a[0], b[0]);
                products(a[1], b[1]);
            }
            fold();
        }
    }
    if constexpr (HAS_SUM) {
        float* __restrict__ out = (OUTS & (F_SQ | F_POW | F_SG)) ? out_sq : out_id;
        out += (int64_t)split * out_stride;
        const int fl = fresh_lane(), ib = i0 + wm * F_T + 4 * (fl >> 4), jb = j0 + wn * F_T + (fl & 15);
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = ib + 16 * m + r;
                if (i < own_i || i >= din) continue;
                float* row = out + (int64_t)i * dout;
#pragma unroll
                for (int n = 0; n < 4; ++n)
                    if (jb + 16 * n >= own_j && jb + 16 * n < dout) row[jb + 16 * n] = sum[m][n][r];
            }
    }
}

template <int OUTS>
hipError_t launch_split(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, const StatPlan& plan, float* out_id,
                        float* out_sq, hipStream_t stream, const float* weight = nullptr, float* norm_partial = nullptr, float alpha = 0.f)
{
    constexpr bool PER_EXAMPLE = !(OUTS == F_PLAIN || OUTS == F_TOKEN);
    const int blocks_m = (int)((din + S_T - 1) / S_T), blocks_n = (int)((dout + S_T - 1) / S_T);
    const int64_t rows_per_split = PER_EXAMPLE ? plan.per_split * T : plan.per_split;
    // rows one descriptor covers: below 2^30 bytes of either operand, whole slabs
    const int window_rows = (int)(((int64_t)1 << 28) / (din > dout ? din : dout) / S_ROWS * S_ROWS);
    const dim3 grid((unsigned)((int64_t)blocks_m * blocks_n * plan.nsplit)), block(S_THREADS);
    stat_f32_split_kernel<OUTS><<<grid, block, 0, stream>>>((const float*)X, (const float*)G, B * T, (int)T, (int)din, (int)dout, rows_per_split,
                                                            window_rows, blocks_m, blocks_n, din * dout, out_id, out_sq, weight, norm_partial, (int)B, alpha);
    return hipGetLastError();
}

}  // namespace

bool f32_split_supports(int64_t B, int64_t T, int64_t din, int64_t dout)
{
    // a width below a block's consists of whole 16-byte chunks; 32-bit byte offsets inside a window of at least 32 rows and
    // inside the rows of a block of S
    if (B * T < 16 || din < 32 || dout < 32 || din > ((int64_t)1 << 20) || dout > ((int64_t)1 << 20)) return false;
    if ((din < S_T && din % 4 != 0) || (dout < S_T && dout % 4 != 0)) return false;
    return f32_split_blocks(din, dout) < ((int64_t)1 << 23);
}

int64_t f32_split_blocks(int64_t din, int64_t dout) { return ((din + S_T - 1) / S_T) * ((dout + S_T - 1) / S_T); }

hipError_t launch_stat_f32_split(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, Mode mode, const StatPlan& plan,
                                 float* out, hipStream_t stream, const float* weight, float* norm_partial, float alpha)
{
    switch (mode) {
    case MODE_IDENTITY: return launch_split<F_PLAIN>(X, G, B, T, din, dout, plan, out, nullptr, stream);
    case MODE_SQUARE: return launch_split<F_SQ>(X, G, B, T, din, dout, plan, nullptr, out, stream);
    case MODE_SIGN: return launch_split<F_SG>(X, G, B, T, din, dout, plan, nullptr, out, stream);
    case MODE_TOKEN_SQ: return launch_split<F_TOKEN>(X, G, B, T, din, dout, plan, out, nullptr, stream);
    case MODE_WEIGHTED: return launch_split<F_IDW>(X, G, B, T, din, dout, plan, out, nullptr, stream, weight);
    case MODE_POWER: return launch_split<F_POW>(X, G, B, T, din, dout, plan, nullptr, out, stream, nullptr, nullptr, alpha);
    case MODE_NORMS: return launch_split<F_NORM>(X, G, B, T, din, dout, plan, nullptr, nullptr, stream, nullptr, norm_partial);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_stat_f32_split_pair(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, const StatPlan& plan,
                                      float* out_id, float* out_sq, hipStream_t stream)
{
    return launch_split<F_ID | F_SQ>(X, G, B, T, din, dout, plan, out_id, out_sq, stream);
}

}  // namespace pex
