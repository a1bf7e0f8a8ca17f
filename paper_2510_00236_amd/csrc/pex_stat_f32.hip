// pex_stat_f32.hip -- fp32 MFMA kernel for S = sum_b phi(X_b^T G_b) and the per-token square, fp32 inputs (gfx950).
//
// Same mathematics as the bf16 kernel (Sec. 2.3): M_b = X_b^T G_b accumulates in registers, phi is applied to the
// finished per-example tile, the per-example gradient never leaves the register file.  fp32 inputs keep true fp32
// products (the 1e-4 tolerance of fp32 inputs forbids rounding them to bf16): v_mfma_f32_16x16x4_f32, 157 TFLOP/s at
// the datasheet clock -- the same as the vector FMA rate with packed operations, which this library is built without.
// Layers large enough run past that rate on the bf16 matrix cores instead (pex_stat_f32_split.hip); this kernel keeps short
// examples, small layers and the statistics that share a contraction with sign.
//
// Bound: the fp32 MFMA pipe, 16 times slower per byte of operand than the bf16 one.  At that ratio the operands need
// no LDS at all: a wave owns a 64 x 64 tile and loads its fragments straight from global memory, so waves share
// nothing, wait for nobody and the kernel has no barrier.  Measured on B=16, T=1024, 1024x4096: phi = square 0.97 ms =
// 142 TFLOP/s, pipes busy 94 % of the cycles.  (Before: 128 x 128 blocks staged through LDS, one barrier per 16 tokens, three
// workgroups per compute unit: 1.18 ms, 76 % -- four waves on four SIMDs that have to meet leave gaps that the other two
// workgroups do not fill.)
//   * The t-major layout is what the MFMA wants: its operand is one float per lane, row (lane % 16) of token
//     (lane / 16).  Rows of the tile may be numbered freely, so operand row p of fragment m is feature 4p + m: the four
//     fragments of a 64-feature panel and four tokens are ONE 16-byte load per lane (16 lanes read 256 contiguous
//     bytes of a token).  Two loads feed 16 MFMAs = 512 cycles.  fp32 rows start at 4-byte boundaries whatever their
//     length, which is all a dwordx4 load asks for, so widths need not be multiples of anything.
//   * The last tile of a width that is no multiple of 64 starts at (width - 64) instead: it overlaps its neighbour and
//     stores only what is its own, so no lane ever reads past the end of a row.
//   * Groups of 4 tokens run through a ring of register sets: the loads of group g + RING - 1 are issued behind the first
//     MFMAs of group g (about RING x 512 cycles of latency covered per wave, times the two waves of a SIMD).  Rows past
//     the end of an example lie outside the buffer descriptor and arrive as zeros; the ring runs on across examples, so
//     an example's first groups are in flight while the previous one is folded.
//
// Several statistics of one call share the contraction: one more register tile of 64 per real-valued statistic, sign counts
// as bytes (16 registers).  What the registers of two waves per SIMD leave is the ring: six groups with two tiles or a tile
// and bytes, four with three tiles, two with all three statistics.  Measured on B=16, T=1024, 1024x4096: identity + square
// 0.98 ms (one after the other 1.92), all three 1.08 ms; three tiles in a ring of six on one wave per SIMD take 1.38 ms, all
// three in a ring of three spill and take 1.29 ms.
#include "pex_f32.h"
#include "pex_internal.h"
#include "pex_tile_map.h"

namespace pex {
namespace {

constexpr int F_ROWS = 4;                  // tokens per group
constexpr int F_THREADS = 256;             // up to four waves: 2 x 2 tiles of 64 x 64
constexpr int F_MAX_U8 = 127;              // examples a byte counter of sign + 1 holds

template <int OUTS, int RING>
__global__ __launch_bounds__(F_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void stat_f32_kernel(
    const float* __restrict__ X, const float* __restrict__ G, int64_t rows_total, int seg_len, int din, int dout, int64_t rows_per_split,
    int window_rows, int waves_n, int blocks_m, int blocks_n, int64_t out_stride, float* __restrict__ out_id, float* __restrict__ out_sq,
    float* __restrict__ out_sg, const float* __restrict__ weight, float* __restrict__ norm_partial, int examples_total, float alpha)
{
    constexpr bool PER_EXAMPLE = !(OUTS == F_PLAIN || OUTS == F_TOKEN);
    constexpr bool HAS_ID = !PER_EXAMPLE || (OUTS & (F_ID | F_IDW)) != 0, HAS_SQ = (OUTS & (F_SQ | F_POW)) != 0, HAS_SG = (OUTS & F_SG) != 0, HAS_SG8 = (OUTS & F_SG8) != 0;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), waves_m = (int)(blockDim.x >> 6) / waves_n;
    int split, bm, bn;
    map_workgroup(blocks_m, blocks_n, split, bm, bn);
    const int own_i = (bm * waves_m + wave / waves_n) * F_T, own_j = (bn * waves_n + wave % waves_n) * F_T;   // first entry that is this tile's own
    if (own_i >= din || own_j >= dout) return;
    const int i0 = own_i + F_T <= din ? own_i : (din > F_T ? din - F_T : 0);
    const int j0 = own_j + F_T <= dout ? own_j : (dout > F_T ? dout - F_T : 0);

    const int64_t row_begin = (int64_t)split * rows_per_split;
    int64_t row_end = row_begin + rows_per_split;
    if (row_end > rows_total) row_end = rows_total;
    const int64_t rows = row_end - row_begin;
    // segment: one example; a plain contraction is folded into its sum every F_CHUNK rows (shorter chains of additions)
    const int slen = PER_EXAMPLE ? seg_len : F_CHUNK;
    const int nst = (slen + F_ROWS - 1) / F_ROWS;
    const int64_t total = PER_EXAMPLE ? rows / seg_len * nst : (rows + F_ROWS - 1) / F_ROWS;

    // operand lane (k, p) = (lane / 16, lane % 16): token k of the group, features 4p .. 4p+3 of the panel (whole chunks: a
    // panel of fewer than 64 features has a multiple of 4 of them)
    const int k = lane >> 4, p = lane & 15;
    const uint32_t xoff = i0 + 4 * p < din ? (uint32_t)(k * din + i0 + 4 * p) * 4u : F_OUTSIDE;
    const uint32_t goff = j0 + 4 * p < dout ? (uint32_t)(k * dout + j0 + 4 * p) * 4u : F_OUTSIDE;

    float4_t acc[4][4], acc_id[HAS_ID ? 4 : 1][4], acc_sq[HAS_SQ ? 4 : 1][4], acc_sg[HAS_SG ? 4 : 1][4];
    uint32_t cnt[HAS_SG8 ? 4 : 1][4];      // four byte counters: sign + 1 of every example added
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            acc[m][n] = float4_t{0.f, 0.f, 0.f, 0.f};
            if (HAS_ID) acc_id[m][n] = acc[m][n];
            if (HAS_SQ) acc_sq[m][n] = acc[m][n];
            if (HAS_SG) acc_sg[m][n] = acc[m][n];
            if (HAS_SG8) cnt[m][n] = 0u;
        }

    // The loads walk through windows: runs of rows of one segment that one pair of descriptors covers, so that a group costs
    // no more than moving the two lane offsets on.  A window ends with its segment (rows past it read as zeros) or where
    // 32-bit offsets would; past the last one the descriptors are empty.
    const float* xbase = X + row_begin * din;
    const float* gbase = G + row_begin * dout;
    const int win_rows = window_rows < slen ? window_rows : slen;      // a multiple of F_ROWS, or the whole segment
    int64_t rows_left = rows;
    int seg_left = slen, win_groups = 0;
    uint32_t xat = xoff, gat = goff;
    const uint32_t xstep = (uint32_t)din * (F_ROWS * 4u), gstep = (uint32_t)dout * (F_ROWS * 4u);
    __amdgpu_buffer_rsrc_t rx, rg;
    auto next_window = [&]() {
        int n = win_rows < seg_left ? win_rows : seg_left;
        if (n > rows_left) n = (int)rows_left;
        rx = __builtin_amdgcn_make_buffer_rsrc((void*)xbase, 0, n * din * 4, 0x00020000);
        rg = __builtin_amdgcn_make_buffer_rsrc((void*)gbase, 0, n * dout * 4, 0x00020000);
        xat = xoff;
        gat = goff;
        xbase += (int64_t)n * din;
        gbase += (int64_t)n * dout;
        rows_left -= n;
        seg_left -= n;
        if (seg_left <= 0) seg_left = slen;
        win_groups = n > 0 ? (n + F_ROWS - 1) / F_ROWS : 1 << 30;
    };
    uint4_t xr[RING], gr[RING];
    auto load_x = [&](int slot) { xr[slot] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)xat, 0, 0); };
    auto load_g = [&](int slot) { gr[slot] = __builtin_amdgcn_raw_buffer_load_b128(rg, (int)gat, 0, 0); };
    auto move_on = [&]() {
        xat += xstep;
        gat += gstep;
        if (--win_groups == 0) next_window();
    };
    // the 16 MFMAs of the group in ring slot `slot`; behind the first of them, the loads into slot `into` (< 0: none).  The
    // column index runs back and forth, so that consecutive MFMAs share an operand register: an MFMA-only loop reaches 155
    // TFLOP/s this way and 147 with two fresh operands at every fourth MFMA.  The fences pin that order.
    auto multiply = [&](int slot, int into) {
        float a[4], b[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            a[e] = __uint_as_float(xr[slot][e]);
            b[e] = __uint_as_float(gr[slot][e]);
            if (OUTS == F_TOKEN) { a[e] *= a[e]; b[e] *= b[e]; }     // exact fp32 squares
        }
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int nn = 0; nn < 4; ++nn) {
                const int n = (m & 1) ? 3 - nn : nn;
                acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m], b[n], acc[m][n], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (into >= 0 && m == 0 && nn == 1) { load_x(into); __builtin_amdgcn_sched_barrier(0); }
                if (into >= 0 && m == 0 && nn == 3) { load_g(into); __builtin_amdgcn_sched_barrier(0); }
                if (into >= 0 && m == 1 && nn == 1) { move_on(); __builtin_amdgcn_sched_barrier(0); }
            }
    };
    int example = (int)(row_begin / seg_len);
    const int ib = i0 + 16 * k, jb = j0 + 4 * p;      // row of (m, r): ib + 4r + m; column of n: jb + n
    auto fold = [&]() {
        float w = 1.f, norm = 0.f;
        if (OUTS & F_IDW) w = weight[example];
        // a norm counts what is this tile's own: not its neighbour's part of an overlapping tile, nothing beyond a narrow panel
        const bool whole = own_i + F_T <= din && own_j + F_T <= dout;
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                uint32_t bytes = 0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float v = acc[m][n][r];
                    if (!PER_EXAMPLE || (OUTS & F_ID)) acc_id[m][n][r] += v;
                    if (OUTS & F_IDW) acc_id[m][n][r] = fmaf(w, v, acc_id[m][n][r]);
                    if (OUTS & F_SQ) acc_sq[m][n][r] = fmaf(v, v, acc_sq[m][n][r]);
                    if (OUTS & F_POW) acc_sq[m][n][r] += power_of(v, alpha);
                    if (OUTS & F_SG) acc_sg[m][n][r] += sign_of(v);
                    if (OUTS & F_SG8) bytes = __builtin_amdgcn_cvt_pk_u8_f32(sign_of(v) + 1.0f, r, bytes);
                    if (OUTS & F_NORM) {
                        const int i = ib + 4 * r + m, j = jb + n;
                        const bool mine = whole || (i >= own_i && i < din && j >= own_j && j < dout);
                        const float u = mine ? v : 0.f;      // (on both factors: an infinity that is not ours times zero is NaN)
                        norm = fmaf(u, u, norm);
                    }
                }
                if (HAS_SG8) cnt[m][n] += bytes;
                acc[m][n] = float4_t{0.f, 0.f, 0.f, 0.f};
            }
        if (OUTS & F_NORM) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) norm += __shfl_xor(norm, off);
            const int tiles_n = (dout + F_T - 1) / F_T;
            if (lane == 0) norm_partial[((int64_t)(own_i / F_T) * tiles_n + own_j / F_T) * examples_total + example] = norm;
        }
        ++example;
    };

    // Whole periods of the ring run without a branch around any load or multiply, so that the compiler can wait for exactly
    // the group it needs (guarded steps made it wait for every load once per period); what is left of a period is
    // already in flight when the loop ends.  Step s refills the slot of step s - 1.
    next_window();
#pragma unroll
    for (int s = 0; s < RING - 1; ++s) {
        load_x(s);
        load_g(s);
        move_on();
        __builtin_amdgcn_sched_barrier(0);
    }
    int st_in_seg = 0;
    auto end_of_step = [&]() {
        if (++st_in_seg == nst) { st_in_seg = 0; fold(); }
    };
    const int64_t periods = total / RING;
    for (int64_t g = 0; g < periods; ++g) {
#pragma unroll
        for (int s = 0; s < RING; ++s) {
            multiply(s, (s + RING - 1) % RING);
            end_of_step();
        }
    }
    const int rest = (int)(total - periods * RING);
#pragma unroll
    for (int s = 0; s < RING - 1; ++s)
        if (s < rest) {
            multiply(s, -1);
            end_of_step();
        }
    if (!PER_EXAMPLE && st_in_seg > 0) fold();
    if (OUTS & F_NORM) return;

    // epilogue: the four column fragments of a lane are four neighbouring columns
    auto store = [&](float* __restrict__ out, auto value) {
        out += (int64_t)split * out_stride;
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = ib + 4 * r + m;
                if (i < own_i || i >= din) continue;
                float* row = out + (int64_t)i * dout;
                const float4_t v = {value(m, 0, r), value(m, 1, r), value(m, 2, r), value(m, 3, r)};
                if (jb >= own_j && jb + 4 <= dout) *(float4_u*)(row + jb) = v;
                else {
#pragma unroll
                    for (int n = 0; n < 4; ++n)
                        if (jb + n >= own_j && jb + n < dout) row[jb + n] = v[n];
                }
            }
    };
    if constexpr (HAS_ID) store(out_id, [&](int m, int n, int r) { return acc_id[m][n][r]; });
    if constexpr (HAS_SQ) store(out_sq, [&](int m, int n, int r) { return acc_sq[m][n][r]; });
    if constexpr (HAS_SG) store(out_sg, [&](int m, int n, int r) { return acc_sg[m][n][r]; });
    if constexpr (HAS_SG8) {
        const int examples = (int)(rows / seg_len);
        store(out_sg, [&](int m, int n, int r) { return (float)((int)((cnt[m][n] >> (8 * r)) & 0xffu) - examples); });
    }
}

template <int OUTS, int RING>
hipError_t launch_f32(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, const StatPlan& plan, float* out_id,
                      float* out_sq, float* out_sg, hipStream_t stream, const float* weight = nullptr, float* norm_partial = nullptr,
                      float alpha = 0.f)
{
    constexpr bool PER_EXAMPLE = !(OUTS == F_PLAIN || OUTS == F_TOKEN);
    int bm, bn;
    f32_tile_shape(din, dout, &bm, &bn);
    const int waves_m = bm / F_T, waves_n = bn / F_T;
    const int blocks_m = (int)((din + bm - 1) / bm), blocks_n = (int)((dout + bn - 1) / bn);
    const int64_t rows_per_split = PER_EXAMPLE ? plan.per_split * T : plan.per_split;
    // rows one descriptor covers: below 2^30 bytes of either operand, whole groups
    int64_t window = ((int64_t)1 << 28) / (din > dout ? din : dout) / F_ROWS * F_ROWS;
    const int window_rows = (int)(window < ((int64_t)1 << 30) ? window : (int64_t)1 << 30);
    const dim3 grid((unsigned)((int64_t)blocks_m * blocks_n * plan.nsplit)), block((unsigned)(waves_m * waves_n * 64));
    stat_f32_kernel<OUTS, RING><<<grid, block, 0, stream>>>((const float*)X, (const float*)G, B * T, (int)T, (int)din, (int)dout, rows_per_split, window_rows, waves_n,
                                                            blocks_m, blocks_n, din * dout, out_id, out_sq, out_sg, weight,
                                                            norm_partial, (int)B, alpha);
    return hipGetLastError();
}

}  // namespace

// Waves of a workgroup: the arrangement of at most four 64 x 64 tiles that makes the fewest workgroups of the layer, among equals
// the one with the fewest waves, then the squarest (2 x 2 draws the fewest bytes).  Workgroups are what counts: a wave without a
// tile exits and leaves its SIMD idle beside the others', and the waves of two small workgroups meet on the same SIMDs.
// Measured, 3 x 52 tiles (152 x 3328, B=22 T=2889 per-token square): 2 x 2 waves 865 us, 1 x 4 609; 2 x 13 tiles (128 x 828, B=32
// T=1997 square): 2 x 1 waves 243 us, 2 x 2 136.
void f32_tile_shape(int64_t din, int64_t dout, int* bm, int* bn)
{
    const int64_t tm = (din + F_T - 1) / F_T, tn = (dout + F_T - 1) / F_T;
    int64_t best = 0;
    int wm = 1, wn = 1;
    for (int a = 1; a <= 4; ++a)
        for (int b = 1; a * b <= 4; ++b) {
            const int64_t blocks = ((tm + a - 1) / a) * ((tn + b - 1) / b);
            const bool better = best == 0 || blocks < best || (blocks == best && (a * b < wm * wn || (a * b == wm * wn && a + b < wm + wn)));
            if (better) { best = blocks; wm = a; wn = b; }
        }
    *bm = wm * F_T;
    *bn = wn * F_T;
}

bool f32_mfma_supports(int64_t B, int64_t T, int64_t din, int64_t dout)
{
    // a panel narrower than a tile must consist of whole 16-byte chunks; the narrowest layers stay on the SIMT kernel
    if (B * T < 16 || din < 32 || dout < 32) return false;
    if ((din < F_T && din % 4 != 0) || (dout < F_T && dout % 4 != 0)) return false;
    // 32-bit byte offsets inside a window of at least four rows
    if (din > ((int64_t)1 << 26) || dout > ((int64_t)1 << 26)) return false;
    // one group of the batch: below 2^31 threads (the planner bounds the groups)
    return ((din + F_T - 1) / F_T) * ((dout + F_T - 1) / F_T) < ((int64_t)1 << 25);
}

int64_t f32_norm_partials(int64_t din, int64_t dout) { return ((din + F_T - 1) / F_T) * ((dout + F_T - 1) / F_T); }

hipError_t launch_stat_f32(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, Mode mode, const StatPlan& plan,
                           float* out, hipStream_t stream, const float* weight, float* norm_partial, float alpha)
{
    if (plan.f32_split) return launch_stat_f32_split(X, G, B, T, din, dout, mode, plan, out, stream, weight, norm_partial, alpha);
    switch (mode) {
    case MODE_IDENTITY: return launch_f32<F_PLAIN, 6>(X, G, B, T, din, dout, plan, out, nullptr, nullptr, stream);
    case MODE_SQUARE: return launch_f32<F_SQ, 6>(X, G, B, T, din, dout, plan, nullptr, out, nullptr, stream);
    case MODE_SIGN: return launch_f32<F_SG, 6>(X, G, B, T, din, dout, plan, nullptr, nullptr, out, stream);
    case MODE_TOKEN_SQ: return launch_f32<F_TOKEN, 6>(X, G, B, T, din, dout, plan, out, nullptr, nullptr, stream);
    case MODE_WEIGHTED: return launch_f32<F_IDW, 6>(X, G, B, T, din, dout, plan, out, nullptr, nullptr, stream, weight);
    case MODE_POWER: return launch_f32<F_POW, 6>(X, G, B, T, din, dout, plan, nullptr, out, nullptr, stream, nullptr, nullptr, alpha);
    case MODE_NORMS: return launch_f32<F_NORM, 6>(X, G, B, T, din, dout, plan, nullptr, nullptr, nullptr, stream, nullptr, norm_partial);
    }
    return hipErrorInvalidValue;
}

bool f32_bytes_suffice(const StatPlan& plan) { return plan.per_split <= F_MAX_U8; }

// Two or three statistics from one contraction; an output that is NULL is not wanted.
hipError_t launch_stat_f32_multi(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, const StatPlan& plan,
                                 float* out_id, float* out_sq, float* out_sg, hipStream_t stream)
{
    if (out_sg && (plan.f32_split || !f32_bytes_suffice(plan))) return hipErrorInvalidValue;
    if (plan.f32_split) return launch_stat_f32_split_pair(X, G, B, T, din, dout, plan, out_id, out_sq, stream);
    if (out_id && out_sq && out_sg) return launch_f32<F_ID | F_SQ | F_SG8, 2>(X, G, B, T, din, dout, plan, out_id, out_sq, out_sg, stream);
    if (out_id && out_sq) return launch_f32<F_ID | F_SQ, 4>(X, G, B, T, din, dout, plan, out_id, out_sq, nullptr, stream);
    if (out_id && out_sg) return launch_f32<F_ID | F_SG8, 6>(X, G, B, T, din, dout, plan, out_id, nullptr, out_sg, stream);
    if (out_sq && out_sg) return launch_f32<F_SQ | F_SG8, 6>(X, G, B, T, din, dout, plan, nullptr, out_sq, out_sg, stream);
    return hipErrorInvalidValue;
}

}  // namespace pex
