// pex_api.hip -- the C ABI of libpex: host-side validation, planning and kernel dispatch.
// Every entry point validates first and launches nothing on error.
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <mutex>

#include "pex_internal.h"

// Scratch of pex_stat_noalloc: device memory that belongs to the library, one copy per GPU, held until the process
// ends.  In host code this name is only a handle for hipGetSymbolAddress; kernels and copies take the address that
// call returns for the current device.
static __device__ __align__(256) unsigned char scratch[PEX_NOALLOC_SCRATCH_BYTES];

namespace pex {

// The address of `scratch` on the current device, looked up once per device.
static hipError_t scratch_address(void** out)
{
    constexpr int MAX_DEVICES = 64;
    static std::mutex mu;
    static void* ptr[MAX_DEVICES] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        ptr[dev] = p;
    }
    *out = ptr[dev];
    return hipSuccess;
}

// Planner options.  Their first values come from the environment, read once per process; afterwards only
// pex_set_option changes them.  Atomics, so a host thread that plans while another one sets an option reads a
// whole value; a plan made under one value and launched under another is caught as PEX_ERR_WORKSPACE.
constexpr int NUM_OPTIONS = 6, PLAN_OPTIONS = 5;       // all; those the plan of a single statistic depends on
constexpr int DEFAULT_OPTIONS[NUM_OPTIONS] = {32, 1, 1, 1, 1, 1};
struct Options {
    std::atomic<int> v[NUM_OPTIONS];
};

static bool known_option(int opt) { return opt >= 0 && opt < NUM_OPTIONS; }

static int clamp_option(int opt, int value)
{
    if (opt == PEX_OPT_MAX_SPLIT) return value < 1 ? 1 : (value > 32 ? 32 : value);
    if (opt == PEX_OPT_GRAM_NORMS) return value < 0 ? 0 : (value > 3 ? 3 : value);   // 2, 3: forced, on small / large blocks
    if (opt == PEX_OPT_STORED_EXAMPLES) return value < 0 ? 0 : (value > 1 ? 1 : value);
    return value < 0 ? 0 : (value > 2 ? 2 : value);      // every other option: 0 = off, 1 = cost model, 2 = forced
}

static Options& options()
{
    static Options o;
    static std::once_flag once;
    std::call_once(once, [] {
        const char* names[NUM_OPTIONS] = {"PEX_MAX_SPLIT", "PEX_TOKEN_PRESQUARE", "PEX_WIDE_BLOCKS", "PEX_GRAM_NORMS", "PEX_MEMORY_FOLD", "PEX_STORED_EXAMPLES"};
        for (int k = 0; k < NUM_OPTIONS; ++k) {
            const char* e = getenv(names[k]);
            o.v[k].store(clamp_option(k, (e && *e) ? atoi(e) : DEFAULT_OPTIONS[k]));
        }
    });
    return o;
}

static int option(int opt) { return options().v[opt].load(); }

// The options one plan is made with: read once, so that a plan is never a mixture.
struct OptionValues {
    int v[PLAN_OPTIONS];
    int operator[](int opt) const { return v[opt]; }
};

static bool stored_examples() { return option(PEX_OPT_STORED_EXAMPLES) != 0; }

// The next number of groups with a smaller largest group (the numbers between share the same plan), past every bound if there is none.
static int64_t more_groups(int64_t units, int64_t ns)
{
    const int64_t per = (units + ns - 1) / ns;
    return per > 1 ? (units + per - 2) / (per - 1) : INT64_MAX;
}

// The bf16 kernels run one workgroup per compute unit, so a launch of `tiles` blocks with the batch in `ns` groups takes
//   rounds(ns) * ceil(units / ns)  unit-times,  rounds = ceil(tiles * ns / 256),
// its workgroups write ns copies of the output (s_bytes each) and the fixed-order reduction reads them back and writes
// the sum, all at ~4 TB/s.
// fold_bytes > 0: every workgroup adds that many bytes to the output in memory after each of its units but the first
// (which stores); the workgroups of a round do so at the same time, and what they move -- read and written back
// across the fabric -- goes at ~5.5 TB/s while they wait (measured: 22 - 29 us for the 67 MB of a 1B-scale layer).
// t_round > 0: what a round costs besides its units (the start of a workgroup).
// Returns the cheapest cost over ns <= max_split and the split that reaches it.
static double cheapest_split(int64_t tiles, int64_t units, double t_unit, double s_bytes, int max_split, int64_t* nsplit, int64_t* per,
                             double fold_bytes = 0.0, double t_round = 0.0)
{
    double best = 0.0;
    const int64_t lim = units < max_split ? units : max_split;
    for (int64_t ns = 1; ns <= lim; ns = more_groups(units, ns)) {
        const int64_t pu = (units + ns - 1) / ns;
        const int64_t ns_eff = (units + pu - 1) / pu;
        const int64_t rounds = (tiles * ns_eff + 255) / 256;
        double cost = (double)rounds * ((double)pu * t_unit + t_round);
        if (fold_bytes > 0.0) {
            const int64_t at_once = tiles * ns_eff < 256 ? tiles * ns_eff : 256;
            cost += (double)rounds * (double)(pu - 1) * (2.0 * (double)at_once * fold_bytes / 5.5e12 + 2.0e-6);
        }
        if (ns_eff > 1) cost += (2 * ns_eff + 1) * s_bytes / 4.0e12 + 3.0e-6;
        if (ns == 1 || cost < best) { best = cost; *nsplit = ns_eff; *per = pu; }
    }
    return best;
}

// The fp32 kernel: a wave multiplies one 64 x 64 tile on the MFMA pipe of its SIMD (0.15e12 FLOP/s; alone there it keeps
// the pipe about 87 % busy, two waves about 95 %), `waves` of them make a workgroup, up to eight waves share a compute unit.
// A group of `pu` units therefore takes as long as the busiest pipe: ceil(workgroups / 256) waves of pu units (the waves of
// workgroups of two or three meet on the same pipes, single waves spread), at least one wave's own work.  Exchange of partial sums as above;
// without any (norms), a round of workgroups costs 1 us.  A unit is whole groups of four rows and, of an example, the fold (`t_fold`).
static double cheapest_split_f32(int64_t tiles, int64_t units, int64_t rows_per_unit, double t_fold, int waves, double s_bytes, int max_split,
                                 int64_t* nsplit, int64_t* per)
{
    double best = 0.0;
    const double wave_unit = 2.0 * (double)((rows_per_unit + 3) / 4 * 4) * 64.0 * 64.0 / 0.15e12 + t_fold;
    const int64_t lim = units < max_split ? units : max_split;
    for (int64_t ns = 1; ns <= lim; ns = more_groups(units, ns)) {
        const int64_t pu = (units + ns - 1) / ns;
        const int64_t ns_eff = (units + pu - 1) / pu;
        const double per_pipe = (double)((tiles * ns_eff + 255) / 256) * (waves > 1 ? 1.0 : 0.25);
        double cost = (double)pu * wave_unit * (per_pipe > 1.0 ? per_pipe * 1.05 : 1.15);
        if (s_bytes == 0.0) cost += (double)((tiles * ns_eff + 255) / 256) * 1.0e-6;
        else if (ns_eff > 1) cost += (2 * ns_eff + 1) * s_bytes / 4.0e12 + 2.5e-6;
        if (ns == 1 || cost < best) { best = cost; *nsplit = ns_eff; *per = pu; }
    }
    return best;
}

// fp32 layers on the bf16 matrix cores: blocks of 128 x 128, two of them on a compute unit.  A slab of 32 tokens takes 1.9 us when
// a block has its unit to itself, two slabs 2.5 us when two blocks share one; the fold of an example 0.6 us (signs and powers 1.3, norms 3.5);
// a launch 8.6 us to start and end (norms 3.8, and 0.3 with every round of blocks).  Partial sums at 6.3 TB/s, 2.4 us for their launch.
// Identity and square together also add S_id up in memory: 64 KiB per block and example, read and written at 4.3 TB/s, of which a seventh of
// the contraction's time is hidden (2048 x 2048, B=32 T=64: 21 us an example; 2048 x 4096, B=8 T=1024: 6 us).  Fitted on 140 drawn
// layers of 8 to 700 us and six statistics: the estimates are within 8 % for four in five, of the pair within 12 %.
static double cheapest_split_f32_pieces(int64_t blocks, int64_t units, int64_t slabs_per_unit, Mode mode, bool pair, double s_bytes, int max_split,
                                        int64_t* nsplit, int64_t* per)
{
    constexpr double SLAB_ALONE = 1.93e-6, SLABS_SHARED = 2.46e-6;
    const bool plain = mode == MODE_IDENTITY || mode == MODE_TOKEN_SQ;
    const double slabs = (double)slabs_per_unit;
    const double t_fold = plain ? 0.1e-6 : mode == MODE_SIGN || mode == MODE_POWER ? 1.33e-6 : mode == MODE_NORMS ? 3.5e-6 : 0.59e-6;
    double best = 0.0;
    const int64_t lim = units < max_split ? units : max_split;
    for (int64_t ns = 1; ns <= lim; ns = more_groups(units, ns)) {
        const int64_t pu = (units + ns - 1) / ns;
        const int64_t ns_eff = (units + pu - 1) / pu;
        const int64_t wgs = blocks * ns_eff, per_cu = (wgs + 255) / 256;
        double t_unit = t_fold;
        if (pair) {
            const double memory = 0.9 * 2.0 * 65536.0 * (double)(wgs < 512 ? wgs : 512) / 3.9e12 - 0.14 * slabs * SLABS_SHARED;
            if (memory > 0.0) t_unit += memory;
        }
        double cost = (double)pu * ((double)(per_cu / 2) * (slabs * SLABS_SHARED + t_unit) + (double)(per_cu % 2) * (slabs * SLAB_ALONE + t_unit));
        cost += mode == MODE_NORMS ? 3.75e-6 + (double)((per_cu + 1) / 2) * 0.3e-6 : 8.6e-6;
        if (mode != MODE_NORMS && ns_eff > 1) cost += (2 * ns_eff + 1) * s_bytes * (pair ? 2.0 : 1.0) / 6.3e12 + 2.35e-6;
        if (ns == 1 || cost < best) { best = cost; *nsplit = ns_eff; *per = pu; }
    }
    return best;
}

// Sustained rate of one compute unit on the bf16 blocks, FLOP/s (measured on Gaussian operands, 1B-scale layers):
// the larger the block, the fewer bytes go from L2 into LDS and from LDS into registers per FLOP.
// chip-wide rates of the two routes to the per-example norms, FLOP/s (measured)
constexpr double GRAM_RATE = 6.0e14, GRAM_STEP = 0.45e-6, GRAM_WIDE_STEP_FULL = 0.9e-6, GRAM_WIDE_STEP = 0.75e-6, DIRECT_NORM_RATE = 1.3e15;

static double bf16_block_rate(int bm, int bn)
{
    const int area = bm * bn;
    return area >= 256 * 256 ? 5.5e12 : (area >= 256 * 192 ? 4.8e12 : 4.3e12);
}

// A unit on a bf16 block, seconds: its slabs of 32 rows and, at the end of an example, the fold into the statistics.  Measured with
// T <= 32 (one slab: 0.45 us on 256 x 128, 0.53 us on 256 x 256), per example: square and weighted sum 1.0 us, power 2.05, identity +
// square 1.2, with signs 1.9, all three 2.3 (256 x 128 blocks); signs 2.95, norms 2.15 (256 x 256).
// Used for the norms and for layers of odd width.  The other plans count the contraction alone: with the fold some layers of few
// examples got up to a fifth slower (and others, of many short ones, a quarter faster).
static double bf16_fold(Mode mode, bool shared, int bm, int bn)
{
    const double fold = shared ? 1.3e-6 : mode == MODE_SIGN ? 1.2e-6 : mode == MODE_NORMS ? 0.8e-6 : mode == MODE_POWER ? 1.6e-6 : 0.55e-6;
    return fold * (bm * bn / 32768.0);
}
static double bf16_unit_with_fold(Mode mode, bool shared, int64_t T, int bm, int bn)
{
    const double slabs = 2.0 * (double)((T + 31) / 32 * 32) * bm * bn / bf16_block_rate(bm, bn);
    return slabs + bf16_fold(mode, shared, bm, bn);
}

// bf16 layers whose rows are not whole 16-byte chunks: padded copies on the MFMA kernels, or the SIMT kernel on the operands as
// they are?  Whichever these estimates say is faster (2500 drawn calls of 8 to 12000 columns, 1 to 600 examples and tokens: chosen
// right but for 2 % of the time; the estimates' own spread is about 10 %).
//
// The SIMT kernel: serial loops of 16 rows on 64 x 64 tiles, 1.4 us a slab plus 0.3 for each workgroup per compute unit, 2.3 us from four on.
static double simt_seconds(int64_t B, int64_t T, int64_t din, int64_t dout, Mode mode)
{
    const bool plain = mode == MODE_IDENTITY || mode == MODE_TOKEN_SQ;
    const int64_t tiles = ((din + 63) / 64) * ((dout + 63) / 64), units = plain ? (B * T + 63) / 64 : B;
    int64_t groups = (1024 + tiles - 1) / tiles;
    if (groups > units) groups = units;
    if (groups > 32) groups = 32;
    const int64_t per = (units + groups - 1) / groups;
    groups = (units + per - 1) / per;
    int64_t steps = per * (plain ? 4 : (T + 15) / 16);
    if (plain && steps > (B * T + 15) / 16) steps = (B * T + 15) / 16;
    const double slabs = (double)steps, density = (double)(tiles * groups) / 256.0;
    double t = slabs * (density < 4.0 ? 1.4e-6 + 0.3e-6 * density : 0.575e-6 * density) + 3.0e-6;
    if (groups > 1 && mode != MODE_NORMS) t += (double)(2 * groups + 1) * (double)din * (double)dout * 4.0 / 4.0e12 + 3.0e-6;
    return t;
}

// The copies: one pass over the operands, the MFMA plan, and about 10 us for two more launches and the start and end of the blocks
// (12: where the two come out alike the SIMT kernel does, which needs no copies).
static double padded_seconds(int64_t B, int64_t T, int64_t width_in, int64_t width_out, Mode mode, bool shared)
{
    const int64_t din = padded_width(width_in), dout = padded_width(width_out);
    const bool plain = mode == MODE_IDENTITY || mode == MODE_TOKEN_SQ, norms = mode == MODE_NORMS;
    int bm, bn;
    bf16_tile_shape(mode, B, &bm, &bn);
    const int64_t tiles = ((din + bm - 1) / bm) * ((dout + bn - 1) / bn), units = plain ? (B * T + 63) / 64 : B;
    const double s_bytes = (double)din * (double)dout * 4.0, rows = (double)B * (double)T;
    const double unit = plain ? 2.0 * 64.0 * bm * bn / bf16_block_rate(bm, bn) : bf16_unit_with_fold(mode, shared, T, bm, bn);
    int64_t ns, per;
    double t = cheapest_split(tiles, units, unit, norms ? 0.0 : s_bytes * (shared ? 2.0 : 1.0), norms ? (B < 1024 ? (int)B : 1024) : 32, &ns, &per, 0.0,
                              norms ? 2.0e-6 : 0.0);
    // per-token square: four such contractions into partial sums of their own, copies of twice the size, seven launches
    if (mode == MODE_TOKEN_SQ)
        return 3.1 * (double)((tiles * ns + 255) / 256) * (double)per * unit + (double)(8 * ns + 1) * s_bytes / 5.0e12 + 10.0 * rows * (double)(din + dout) / 15.0e12 + 36.0e-6;
    if (mode == MODE_SIGN && bm == 256 && bn == 256) {       // partial counts as bytes
        const double bytes = cheapest_split(tiles, units, unit, (double)sign_byte_partial_bytes(din, dout), 32, &ns, &per);
        if (bytes < t) t = bytes;
    }
    return t + 4.0 * rows * (double)((width_in % 8 != 0 ? din : 0) + (width_out % 8 != 0 ? dout : 0)) / 5.0e12 + 12.0e-6;
}

// `passes` = statistics the SIMT kernel would make one by one
static bool padding_pays(int64_t B, int64_t T, int64_t din, int64_t dout, Mode mode, int passes)
{
    if (din % 8 == 0 && dout % 8 == 0) return false;
    if (!pad_supports(B * T, din, dout) || !bf16_supports(B, T, padded_width(din), padded_width(dout))) return false;
    return padded_seconds(B, T, din, dout, mode, passes > 1) < simt_seconds(B, T, din, dout, mode) * passes;
}

// The partial sums of an fp32 call that pex_stat_noalloc has always had room for, by the shape alone: those of as many groups as
// put three workgroups of 128 x 128 on every compute unit, or four of 64 x 64 where rows are not whole 16-byte chunks.  A layer
// within the scratch by this figure keeps a plan that fits it.
static size_t scratch_charge_f32(int64_t B, int64_t T, int64_t din, int64_t dout, Mode mode, int max_split)
{
    const bool chunked = din % 4 == 0 && dout % 4 == 0 && din >= 32 && dout >= 32 && B * T >= 16;
    const int64_t edge = chunked ? 128 : 64, target = chunked ? 768 : 1024;
    const int64_t tiles = ((din + edge - 1) / edge) * ((dout + edge - 1) / edge);
    const int64_t units = mode == MODE_IDENTITY ? (B * T + 63) / 64 : B;
    int64_t ns = (target + tiles - 1) / tiles;
    if (ns > max_split) ns = max_split;
    if (ns > units) ns = units;
    const int64_t per = (units + ns - 1) / ns;
    ns = (units + per - 1) / per;
    return ns > 1 ? (size_t)ns * (size_t)din * (size_t)dout * sizeof(float) : 0;
}

static StatPlan make_large_plan(int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt, Mode mode, bool allow_wide, bool allow_pad,
                          const OptionValues& options)
{
    StatPlan p{};
    p.out_rows = din;
    p.out_cols = dout;
    // (a plan on one block shape is one of several statistics at once; option 0: squares inside the contraction, of odd widths the
    // SIMT kernel's)
    if (mode == MODE_TOKEN_SQ && options[PEX_OPT_TOKEN_PRESQUARE] == 0) allow_pad = false;
    if (allow_pad && dt == PEX_BF16 && padding_pays(B, T, din, dout, mode, allow_wide ? 1 : 2)) {
        p.square_halves = mode == MODE_TOKEN_SQ;
        p.copy_x = din % 8 != 0 || p.square_halves;
        p.copy_g = dout % 8 != 0 || p.square_halves;
        din = padded_width(din);
        dout = padded_width(dout);
    }
    p.din = din;
    p.dout = dout;
    const bool padded = din != p.out_rows || dout != p.out_cols;
    const bool per_example = (mode == MODE_SQUARE || mode == MODE_SIGN || mode == MODE_NORMS || mode == MODE_WEIGHTED || mode == MODE_POWER);
    p.kernel = (dt == PEX_BF16 && bf16_supports(B, T, din, dout)) ? 1 : 0;
    if (dt == PEX_F32 && f32_mfma_supports(B, T, din, dout)) p.kernel = 2;

    // The unit the batch axis is split in: whole examples when phi is applied per example (the sum over
    // the sequence must be complete before phi), slabs of 64 rows of the flattened [B*T] axis otherwise.
    int64_t tiles, target, units;
    int bm = 64, bn = 64;
    if (p.kernel == 1) {
        bf16_tile_shape(mode, B, &bm, &bn);
        target = 256;    // one workgroup per compute unit
    } else if (p.kernel == 2) {
        f32_tile_shape(din, dout, &bm, &bn);
        target = 0;      // by cost model
    } else {
        target = 1024;   // four small workgroups per compute unit
    }
    tiles = ((din + bm - 1) / bm) * ((dout + bn - 1) / bn);
    const int64_t slab = 64;
    units = per_example ? B : (B * T + slab - 1) / slab;
    // The option bounds the workspace; the norms exchange no partial sums, so unless it is lowered they take as many groups as
    // there are examples (B=56 T=1150 64x312, two blocks: 32 groups 71 us, 56 groups 27)
    int max_split = options[PEX_OPT_MAX_SPLIT];
    if (mode == MODE_NORMS && max_split == 32) max_split = B < 1024 ? (int)B : 1024;
    if (p.kernel != 0) {
        // the MFMA kernels put blocks and groups in one grid dimension, which holds fewer than 2^32 threads (the SIMT kernel has
        // a dimension for each)
        const int64_t threads = p.kernel == 2 ? (int64_t)(bm / 64) * (bn / 64) * 64 : 512;
        const int64_t fit = (((int64_t)1 << 32) - 1) / (tiles * threads);
        if (max_split > fit) max_split = fit < 1 ? 1 : (int)fit;
    }
    int64_t nsplit = 1, per = units;
    double best_bf16 = 0.0;
    int64_t wide_cols = 0, wide_nsplit = 1, wide_per = units, direct_nsplit = 1;
    bool sign_bytes = false, mem_fold = false;
    if (p.kernel == 2) {
        // Calls that pex_stat_noalloc has always taken keep their partial sums within its scratch; the others are free (B=42 T=112 704x3648
        // sign, 10 MB of S, three groups in 32 MB: 321 us, free 311; B=16 T=512 1536x1536 square 369 and 319)
        const bool held = mode <= MODE_SIGN && scratch_charge_f32(B, T, din, dout, mode, max_split) <= (size_t)PEX_NOALLOC_SCRATCH_BYTES;
        const int64_t fit = (int64_t)PEX_NOALLOC_SCRATCH_BYTES / (din * dout * 4);
        // folds as measured on one wave per SIMD (T=1 .. 128, 2048 x 2048), seconds per example: with them left out, layers of a few
        // tokens per example were planned in one group (B=72 T=1 880x128 power 83 us, 17 with them; B=26 T=1 118x384 sign 39 and 12)
        const double t_fold = !per_example ? 0.0 : !allow_wide ? 1.0e-6 : mode == MODE_SIGN ? 1.07e-6 : mode == MODE_NORMS ? 1.15e-6 :
                              mode == MODE_POWER ? 0.88e-6 : 0.3e-6;
        const double s_bytes = mode == MODE_NORMS ? 0.0 : (double)din * (double)dout * 4.0;
        const int most = !held || fit > max_split ? max_split : (fit < 1 ? 1 : (int)fit);
        const double direct = p.seconds = cheapest_split_f32(tiles, units, per_example ? T : slab, t_fold, (bm / 64) * (bn / 64), s_bytes, most, &nsplit, &per);
        // ... or split into bf16 pieces, where that is faster (never for examples of fewer than 48 tokens, a slab and a half: not compared)
        if (allow_pad && f32_split_supports(B, T, din, dout) && (per_example ? T : B * T) >= 48) {
            int64_t ns_p = 1, per_p = units;
            const int64_t blocks = f32_split_blocks(din, dout), fit_p = (((int64_t)1 << 32) - 1) / (blocks * 256);
            const double pieces = cheapest_split_f32_pieces(blocks, units, ((per_example ? T : slab) + 31) / 32, mode, !allow_wide, s_bytes,
                                                            most > fit_p ? (int)fit_p : most, &ns_p, &per_p);
            p.seconds = pieces < direct ? pieces : direct;
            if (pieces < direct) {
                p.f32_split = true;
                direct_nsplit = nsplit;
                nsplit = ns_p;
                per = per_p;
            }
        }
    } else if (p.kernel != 1) {
        nsplit = (target + tiles - 1) / tiles;
        if (nsplit > max_split) nsplit = max_split;
        if (nsplit > units) nsplit = units;
        if (nsplit < 1) nsplit = 1;
        per = (units + nsplit - 1) / nsplit;
        p.seconds = simt_seconds(B, T, din, dout, mode) * (allow_wide ? 1.0 : 2.0);
    } else {
        // A unit-time is one example (or 64 rows) on one block.
        const double rows_per_unit = per_example ? (double)T : (double)slab;
        const bool folds = per_example && (padded || mode == MODE_NORMS);
        const double t_unit = folds ? bf16_unit_with_fold(mode, !allow_wide, T, bm, bn) : 2.0 * rows_per_unit * bm * bn / bf16_block_rate(bm, bn);
        // (the per-example norms exchange no partial sums of S, only one number per workgroup and example: without the cost of a round
        // they would take every group there is to save a fraction of one; B=131 T=67 10304x64, 41 blocks: 6 groups 77 us, 131 125)
        double best = cheapest_split(tiles, units, t_unit, mode == MODE_NORMS ? 0.0 : (double)din * (double)dout * 4.0, max_split, &nsplit, &per, 0.0,
                                     mode == MODE_NORMS ? 2.0e-6 : 0.0);
        // Packed sign counts can be exchanged as bytes while a group holds at most 127 examples: a quarter of the
        // traffic, so more groups pay.  Planned with that cost; kept if the groups it gives are small enough.
        if (mode == MODE_SIGN && bm == 256 && bn == 256) {
            int64_t ns_b = 1, per_b = units;
            const double cost_b = cheapest_split(tiles, units, t_unit, (double)sign_byte_partial_bytes(din, dout), max_split, &ns_b, &per_b);
            if (ns_b > 1 && sign_byte_partials_possible(B, per_b) && cost_b <= best) {
                best = cost_b;
                nsplit = ns_b;
                per = per_b;
                sign_bytes = true;
            }
        }
        // One statistic on two register tiles may put its first columns on the wider block (256 x 192) and only the
        // remaining columns on the 256 x 128 block, each part with a split of the batch of its own.  Candidates: every
        // number of wide block columns up to 64, beyond that the largest number that fits k rounds of 256 workgroups,
        // and all columns wide.
        const int wide_opt = options[PEX_OPT_WIDE_BLOCKS];
        if (allow_wide && wide_opt != 0 && (mode == MODE_SQUARE || mode == MODE_WEIGHTED || mode == MODE_POWER) && bm == 256 && bn == 128) {
            int wm, wn;
            bf16_wide_tile_shape(&wm, &wn);
            const int64_t tiles_m = (din + wm - 1) / wm, max_wide = dout / wn;
            const double t_wide = folds ? bf16_unit_with_fold(mode, false, T, wm, wn) : 2.0 * (double)T * wm * wn / bf16_block_rate(wm, wn);
            auto consider = [&](int64_t na, bool forced) {
                const int64_t rest = dout - na * wn;
                int64_t ns_w = 1, per_w = units, ns_r = 1, per_r = units;
                double cost = cheapest_split(tiles_m * na, units, t_wide, (double)din * (double)(na * wn) * 4.0, max_split, &ns_w, &per_w);
                if (rest > 0)
                    cost += 5.0e-6 + cheapest_split(tiles_m * ((rest + bn - 1) / bn), units, t_unit, (double)din * (double)rest * 4.0, max_split,
                                                    &ns_r, &per_r);
                if (forced || cost < best) {
                    best = cost;
                    wide_cols = na * wn;
                    wide_nsplit = (units + per_w - 1) / per_w;
                    wide_per = per_w;
                    nsplit = ns_r;
                    per = per_r;
                }
            };
            for (int64_t na = 1; na <= max_wide && na <= 64; ++na) consider(na, false);
            for (int64_t k = 1; k <= 64 && max_wide > 64; ++k) {
                const int64_t na = (256 * k) / tiles_m;
                if (na > 64 && na < max_wide) consider(na, false);
            }
            if (max_wide > 64) consider(max_wide, false);
            if (wide_opt == 2 && max_wide >= 1) consider(max_wide, true);      // forced: as many wide block columns as fit
        }
        // ... or keep no second register tile at all: 256 x 256 blocks (eight waves: 5.2e12 FLOP/s per compute unit) that
        // add phi(M_b) to the output in memory at the end of every example
        const int fold_opt = options[PEX_OPT_MEMORY_FOLD];
        if (allow_wide && fold_opt != 0 && (mode == MODE_SQUARE || mode == MODE_WEIGHTED || mode == MODE_POWER) && bm == 256 && bn == 128 &&
            dout < ((int64_t)1 << 20)) {      // 32-bit byte offsets inside a tile of the output
            int fm, fn;
            bf16_tile_shape(MODE_IDENTITY, B, &fm, &fn);
            const int64_t tiles_f = ((din + fm - 1) / fm) * ((dout + fn - 1) / fn);
            int64_t ns_f = 1, per_f = units;
            const double cost = cheapest_split(tiles_f, units, 2.0 * (double)T * fm * fn / 5.2e12, (double)din * (double)dout * 4.0, max_split,
                                               &ns_f, &per_f, (double)fm * fn * 4.0);
            if (fold_opt == 2 || cost < best) {
                best = cost;
                mem_fold = true;
                wide_cols = 0;
                wide_nsplit = 1;
                nsplit = ns_f;
                per = per_f;
            }
        }
        best_bf16 = best;
    }
    nsplit = (units + per - 1) / per;      // no empty group
    if (p.kernel == 1) {
        p.seconds = padded ? padded_seconds(B, T, p.out_rows, p.out_cols, mode, !allow_wide) : best_bf16;
        if (!padded && mode != MODE_NORMS) {      // what the plan is chosen without: folds, the start and end of a launch, the launch of the sum
            p.seconds += 5.0e-6 + (nsplit > 1 ? 4.5e-6 : 0.0);
            if (per_example && !mem_fold) {
                const int64_t rest = dout - wide_cols, rounds = (((din + bm - 1) / bm) * ((rest + bn - 1) / bn) * nsplit + 255) / 256;
                p.seconds += (double)(rounds * per) * bf16_fold(mode, !allow_wide, bm, bn);
            }
        }
    }
    p.nsplit = (int)nsplit;
    p.per_split = per_example ? per : per * slab;
    // Per-token square on the MFMA kernel: squaring the operands inside the kernel (global -> registers -> LDS instead
    // of direct-to-LDS loads) costs about +42 % time; squaring them once into bf16 copies costs one
    // pass over X and G at HBM speed (~5.5 TB/s, 4 bytes moved per element).  The copies win when din*dout/(din+dout)
    // is large.  Measured, inside and by copies, us: 32 x 1024 tokens, 1280x5120 464, 503; 16 x 1024, 1536x6144 348, 344;
    // 16 x 1024, 2048x4096 270, 261; 16 x 2048, 2048x8192 963, 925.
    const int presquare = options[PEX_OPT_TOKEN_PRESQUARE];
    if (mode == MODE_TOKEN_SQ && p.kernel == 1 && presquare != 0 && !p.square_halves) {
        const double elems = (double)B * (double)T * (double)(din + dout);
        const double t_pre = 4.0 * elems / 5.5e12 + 6.0e-6;
        const double t_fused_extra = 0.42 * 2.0 * (double)B * (double)T * (double)din * (double)dout / 1.3e15;
        if (t_pre < t_fused_extra || presquare == 2) p.copy_x = p.copy_g = true;
    }
    const size_t copied = (p.copy_x ? (size_t)din : 0) + (p.copy_g ? (size_t)dout : 0);
    p.copy_bytes = ((size_t)B * (size_t)T * copied * (p.square_halves ? 4 : 2) + 255) & ~(size_t)255;
    p.sign_bytes = sign_bytes && nsplit > 1;
    p.mem_fold = mem_fold;
    p.wide_cols = wide_cols;
    p.wide_nsplit = (int)wide_nsplit;
    p.wide_per_split = wide_per;
    p.wide_ws_bytes = (wide_cols > 0 && wide_nsplit > 1) ? (size_t)wide_nsplit * (size_t)din * (size_t)wide_cols * sizeof(float) : 0;
    p.ws_bytes = p.copy_bytes + p.wide_ws_bytes +
                 ((nsplit > 1 && dout > wide_cols) ? (size_t)nsplit * (size_t)din * (size_t)(dout - wide_cols) * sizeof(float) : 0);
    if (p.square_halves) p.ws_bytes = p.copy_bytes + (size_t)4 * (size_t)nsplit * (size_t)din * (size_t)dout * sizeof(float);
    if (p.sign_bytes) p.ws_bytes = p.copy_bytes + (size_t)nsplit * sign_byte_partial_bytes(din, dout);
    if (mode == MODE_NORMS) {   // no S at all: one partial of ||M_b||^2 per tile (and wave) and example
        const int64_t nparts = p.kernel == 1 ? bf16_norm_partials(din, dout) : p.kernel == 2 ? (p.f32_split ? 4 * f32_split_blocks(din, dout) : f32_norm_partials(din, dout)) : generic_norm_partials(din, dout);
        p.ws_bytes = p.copy_bytes + (size_t)nparts * (size_t)B * sizeof(float);
        // Through the Gram matrices instead: 2 T^2 (din + dout) FLOP per example (a little over half of it with the
        // symmetry, in 128 x 128 blocks) against 2 T din dout, on a kernel of lower rate but with one workgroup per block
        // and example -- no batch split, however few tiles the layer has.
        // Not for padded copies: layers of odd width keep the contraction.  A sum of squares is exact to rounding whatever the inputs,
        // <X X^T, G G^T> cancels where tokens are alike (X = 1 + 0.03 noise, G of zero mean over the tokens, B=4 T=190 257x40: relative
        // error 2e-8 by the contraction, 5e-5 through the Gram matrices).
        const int gram_opt = options[PEX_OPT_GRAM_NORMS];
        if (dt == PEX_BF16 && gram_opt != 0 && p.copy_bytes == 0 && gram_supports(B, T, din, dout)) {
            // Gram kernel: 6.0e14 FLOP/s on a full chip (its 128 x 128 blocks draw twice the bytes per FLOP from L2 that
            // the 256 x 256 blocks of the contraction do), and never faster than its serial loop over the features, one
            // 64-feature step per ~0.45 us (measured with fewer workgroups than compute units).  Contraction: the plan's
            // rounds, plus ~20 us of start-up, epilogue and reduction on small layers.
            const double steps = (double)((din + 63) / 64 + (dout + 63) / 64);
            double t_gram = 2.0 * (double)B * (double)gram_norm_partials(T) * 128.0 * 128.0 * (double)(din + dout) / GRAM_RATE;
            if (t_gram < steps * GRAM_STEP) t_gram = steps * GRAM_STEP;
            t_gram += 6.0e-6;
            double t_direct = 2.0 * (double)B * (double)T * (double)din * (double)dout / DIRECT_NORM_RATE;
            if (p.kernel == 1) {
                const double t_unit = 2.0 * (double)T * bm * bn / bf16_block_rate(bm, bn);
                const double t_rounds = (double)((tiles * p.nsplit + 255) / 256) * (double)((B + p.nsplit - 1) / p.nsplit) * t_unit;
                if (t_rounds > t_direct) t_direct = t_rounds;
            }
            t_direct += 20.0e-6;
            // On 256 x 256 blocks: half the bytes per FLOP; one workgroup per block and example in rounds of 256, each a
            // serial loop of 32-feature steps (measured: ~0.9 us per step on a full chip, ~0.75 us below that), and the
            // parked blocks written and read once (~4 TB/s); while they stay below a quarter of a GiB.
            const size_t park = gram_wide_park_bytes(B, T);
            const double steps_w = (double)((din + 31) / 32 + (dout + 31) / 32);
            const int64_t wgs = B * gram_wide_partials(T);
            double t_wide = (double)((wgs + 255) / 256) * steps_w * (wgs > 256 ? GRAM_WIDE_STEP_FULL : GRAM_WIDE_STEP);
            t_wide += 2.0 * (double)park / 4.0e12 + 8.0e-6;
            const bool wide_ok = park <= ((size_t)256 << 20);
            if (gram_opt == 3 ? wide_ok : (gram_opt == 1 && wide_ok && t_wide < t_gram && t_wide < t_direct)) {
                p.gram = p.gram_wide = true;
                p.seconds = t_wide;
                p.ws_bytes = p.copy_bytes + (((size_t)gram_wide_partials(T) * (size_t)B * sizeof(float) + 255) & ~(size_t)255) + park;
            } else if (gram_opt == 2 || gram_opt == 3 || t_gram < t_direct) {
                p.gram = true;
                p.seconds = t_gram;
                p.ws_bytes = p.copy_bytes + (size_t)gram_norm_partials(T) * (size_t)B * sizeof(float);
            }
        }
    }
    p.query_bytes = p.ws_bytes;
    if (p.f32_split && mode != MODE_NORMS && direct_nsplit > nsplit) p.query_bytes = (size_t)direct_nsplit * (size_t)din * (size_t)dout * sizeof(float);
    return p;
}

// The kernel of small layers: eight waves a workgroup, one workgroup a compute unit.  A wave's step (32 tokens of bf16, 16 of fp32) takes
// 1.04 us and 2.1 where the waves divide an example's tokens, 0.85 and 1.95 where they divide the examples (fp32: the MFMA pipe, two
// waves on each; identity and square together on tiles of half the width 0.75 and 1.1), the end of an example 0.45 us (1.0 of a norm or a
// plain contraction); a launch 3 to 4 us to start and end, another round of workgroups 3, the sum of the norms' parts 2.5.  Every tile reads its features of all tokens: 128-byte lines, one more where rows do not start at
// one, at 14 TB/s from the caches; operands that an XCD's cache does not hold come once for each of up to eight of them at 6.5 TB/s.  That is
// the bound of layers of some dozen tiles with many tokens (110 x 535 tokens, 328 x 350: 105 us, planned at 44 without it, and 62 by
// padded copies).  Stores of 16 bytes at 4 TB/s, partial sums at 5, 4 us for their launch.  Fitted on 260 drawn layers, five
// statistics, both ways to divide the work: estimates within 20 % for four in five.
static double cheapest_small(int64_t din, int64_t dout, int64_t rows, int64_t units, int64_t rows_per_unit, bool bf16, Mode mode, bool pair, int kw,
                             int64_t* nsplit, int64_t* per)
{
    const bool plain = mode == MODE_IDENTITY || mode == MODE_TOKEN_SQ, norms = mode == MODE_NORMS;
    const bool half = pair && kw == 1;
    const int64_t tiles = small_tiles(din, dout, half), rows_per_step = bf16 ? 32 : 16, size = bf16 ? 2 : 4;
    const double t_step = kw == 8 ? (bf16 ? 1.04e-6 : 2.1e-6) : half ? (bf16 ? 0.75e-6 : 1.1e-6) : (bf16 ? 0.85e-6 : 1.95e-6);
    const double t_fold = plain || (norms && kw == 1) ? 1.0e-6 : 0.45e-6;
    const double start = (plain ? 3.0e-6 : kw == 1 ? 4.0e-6 : 3.4e-6) + (norms ? 2.5e-6 : pair ? 0.6e-6 : 0.0), next_round = 3.0e-6;
    auto lines = [&](int64_t width, int64_t cols) { return (double)(cols * size) / 128.0 + (width * size % 128 != 0 ? 0.9 : 0.0); };
    const double caches = (double)tiles * (double)rows * (lines(din, 64) + lines(dout, half ? 32 : 64)) * 128.0 / 14.0e12, c2 = caches * caches;
    const double x_bytes = (double)(rows * din * size), g_bytes = (double)(rows * dout * size);
    const int64_t tiles_m = (din + 63) / 64, tiles_n = tiles / tiles_m;
    const bool fits = x_bytes + g_bytes <= 32.0e6;
    const double misses = (x_bytes * (double)(fits ? 1 : tiles_n < 8 ? tiles_n : 8) + g_bytes * (double)(fits ? 1 : tiles_m < 8 ? tiles_m : 8)) / 6.5e12,
                 m2 = misses * misses;
    const double s_bytes = norms ? 0.0 : (double)din * (double)dout * (pair ? 8.0 : 4.0);
    const int64_t most = norms ? 1024 : 32, lim = units < most ? units : most;
    double best = 0.0;
    for (int64_t ns = 1; ns <= lim; ns = more_groups(units, ns)) {
        const int64_t pu = (units + ns - 1) / ns;
        const int64_t ns_eff = (units + pu - 1) / pu;
        const int64_t rounds = (tiles * ns_eff + 255) / 256;
        double unit;
        if (plain) {
            const int64_t own = pu * rows_per_unit, steps = ((own + 7) / 8 + rows_per_step - 1) / rows_per_step;
            unit = (double)steps * t_step + (double)((own + 8191) / 8192) * t_fold;
        } else {
            const int64_t steps = (rows_per_unit + rows_per_step - 1) / rows_per_step;
            unit = kw == 1 ? (double)((pu + 7) / 8) * ((double)steps * t_step + t_fold) : (double)pu * ((double)((steps + 7) / 8) * t_step + t_fold);
        }
        const double waves = (double)rounds * unit, w2 = waves * waves;
        double cost = sqrt(sqrt(w2 * w2 + c2 * c2 + m2 * m2)) + start + (double)(rounds - 1) * next_round + s_bytes / 4.0e12;       // the largest of the three, and more where they are alike
        if (!norms && ns_eff > 1) cost += (double)(2 * ns_eff) * s_bytes / 5.0e12 + 4.0e-6;
        if (ns == 1 || cost < best) { best = cost; *nsplit = ns_eff; *per = pu; }
    }
    return best;
}

// The kernel of small layers where its estimate is the lowest.  The options choose among the other kernels: a layer planned under one
// that is not at its default stays on them.
static StatPlan make_plan(int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt, Mode mode, bool allow_wide, bool allow_pad, bool allow_small,
                          const OptionValues& options)
{
    if (mode == MODE_NORMS && options[PEX_OPT_MAX_SPLIT] < 32) {
        // the same bits under every bound on the groups: by the same route and kernel, in no more groups
        OptionValues unbound = options;
        unbound.v[PEX_OPT_MAX_SPLIT] = 32;
        StatPlan p = make_plan(B, T, din, dout, dt, mode, allow_wide, allow_pad, allow_small, unbound);
        const int64_t most = options[PEX_OPT_MAX_SPLIT];
        if (!p.gram && p.nsplit > most) {
            p.per_split = (B + most - 1) / most;
            p.nsplit = (int)((B + p.per_split - 1) / p.per_split);
        }
        return p;
    }
    StatPlan p = make_large_plan(B, T, din, dout, dt, mode, allow_wide, allow_pad, options);
    // (What calls of 10 to 200 us take of the large plans' estimates, in the median: bf16 layers 0.8, on the SIMT kernel 0.88; norms by
    // the contraction 0.75, of padded copies 0.67, by Gram matrices 0.97, on the SIMT kernel 1.1; the fp32 kernel 3 us more but for the norms.)
    const bool norms = mode == MODE_NORMS, pair = !allow_wide, copies = p.kernel == 1 && p.copy_bytes > 0;       // pair: identity and square together
    if (dt == PEX_BF16) p.seconds *= p.kernel == 0 ? (norms ? 1.1 : 0.88) : !norms ? 0.8 : copies ? 0.67 : p.gram ? 0.97 : 0.75;
    else if (p.kernel == 2 && !p.f32_split && !norms) p.seconds += 3.0e-6;
    // (a step is 32 or 16 tokens: examples of one to three would be nearly all padding.  Of layers with more tiles than these the large
    // kernels' estimates are too high, by 30 % for norms at half a chip: norms 46 us there and 85 here, signs 66 and 98 at 640 tiles,
    // but squares 113 and 66; more than 1024 were not compared)
    const int64_t most_tiles = mode == MODE_NORMS ? 128 : mode == MODE_SIGN ? 256 : 1024;
    if (!allow_pad || !allow_small || T < 4 || small_tiles(din, dout) > most_tiles || !small_supports(T, din, dout, dt, mode)) return p;
    for (int k = 0; k < PLAN_OPTIONS; ++k)
        if (options[k] != DEFAULT_OPTIONS[k]) return p;
    const bool plain = mode == MODE_IDENTITY || mode == MODE_TOKEN_SQ;
    const int64_t units = plain ? (B * T + 63) / 64 : B;
    StatPlan s{};
    s.seconds = 1.0;
    for (const int kw : {1, 8}) {
        if (plain && kw == 1) continue;
        int64_t ns = 1, per = units;
        const double t = cheapest_small(din, dout, B * T, units, plain ? 64 : T, dt == PEX_BF16, mode, pair, kw, &ns, &per);
        if (t < s.seconds) {
            s.seconds = t;
            s.small_kw = kw;
            s.nsplit = (int)ns;
            s.per_split = plain ? per * 64 : per;
        }
    }
    // (Of 211 bf16 and 49 fp32 layers and five statistics the choice is 1.3 % slower in the mean than the better kernel every time, and four of
    // 1100 calls are slower than without the kernel by more than 6 %, at most 34 %.  Norms that would go by the contraction on whole chunks
    // leave it for a clear gain only.)
    const double margin = norms && dt == PEX_BF16 && p.kernel == 1 && !copies && !p.gram && s.seconds >= 15.0e-6 ? 1.6 : 1.05;
    if (s.seconds * margin >= p.seconds) return p;
    s.kernel = p.kernel;
    s.out_rows = s.din = din;
    s.out_cols = s.dout = dout;
    s.wide_nsplit = 1;
    s.wide_per_split = B;
    s.ws_bytes = mode == MODE_NORMS ? (size_t)small_tiles(din, dout) * s.small_kw * B * sizeof(float)
                 : s.nsplit > 1     ? (size_t)s.nsplit * (size_t)din * (size_t)dout * sizeof(float) : 0;
    s.query_bytes = s.ws_bytes > p.query_bytes ? s.ws_bytes : p.query_bytes;
    return s;
}

// A plan is a function of the shape, the statistic and the options; weighing the candidates takes 1 to 4 us, as long as a
// launch, and up to 12 for the norms of a thousand examples.  Each host thread keeps sixteen, one per hash of what they depend on.
StatPlan plan_stat(int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt, Mode mode, bool allow_wide, bool allow_pad, bool allow_small)
{
    struct Kept {
        int64_t key[5];
        OptionValues options;
        bool valid;
        StatPlan plan;
    };
    static thread_local Kept kept[16] = {};
    Kept now{};
    now.key[0] = B;
    now.key[1] = T;
    now.key[2] = din;
    now.key[3] = dout;
    now.key[4] = (int64_t)dt * 64 + (int64_t)mode * 8 + (allow_small ? 4 : 0) + (allow_wide ? 2 : 0) + (allow_pad ? 1 : 0);
    uint64_t h = 0;
    for (const int64_t k : now.key) h = (h ^ (uint64_t)k) * 0x9e3779b97f4a7c15ull;
    bool same = true;
    Kept& at = kept[h >> 60];
    for (int k = 0; k < PLAN_OPTIONS; ++k) {
        now.options.v[k] = option(k);
        same = same && now.options[k] == at.options[k];
    }
    for (int k = 0; k < 5; ++k) same = same && now.key[k] == at.key[k];
    if (at.valid && same) return at.plan;
    now.plan = make_plan(B, T, din, dout, dt, mode, allow_wide, allow_pad, allow_small, now.options);
    now.valid = true;
    at = now;
    return now.plan;
}

// The plan of a call that has `bytes` of workspace: a layer that does not fit with the kernel of small layers goes without it, one whose
// padded copies do not fit, or that does not with bf16 pieces, runs on the operands as they are.  A call that fits none gets the first plan.
static StatPlan plan_within(int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt, Mode mode, size_t bytes)
{
    const StatPlan first = plan_stat(B, T, din, dout, dt, mode);
    StatPlan plan = first;
    if (plan.query_bytes > bytes && plan.small_kw > 0) plan = plan_stat(B, T, din, dout, dt, mode, true, true, false);
    if (plan.query_bytes > bytes && (plan.din != din || plan.dout != dout || plan.f32_split)) plan = plan_stat(B, T, din, dout, dt, mode, true, false);
    return plan.query_bytes <= bytes ? plan : first;
}

static pex_status check_stat_args(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout,
                                  pex_dtype dt, const float* S)
{
    if (!X || !G || !S) return PEX_ERR_NULL;
    if (dt != PEX_F32 && dt != PEX_BF16) return PEX_ERR_DTYPE;
    if (B < 1 || T < 1 || din < 1 || dout < 1) return PEX_ERR_SHAPE;
    const int64_t lim = (int64_t)1 << 31;
    if (din >= lim || dout >= lim || B >= lim || T >= lim || B * T >= lim) return PEX_ERR_SHAPE;
    if (((uintptr_t)X | (uintptr_t)G | (uintptr_t)S) & 15u) return PEX_ERR_ALIGN;
    // Largest din of the layers that are not whole 16-byte chunks of a row or too small for the MFMA kernels (the SIMT kernel
    // puts the tiles of din, 64 rows, in the second grid dimension), and of the other fp32 layers.
    const int64_t chunk = dt == PEX_BF16 ? 8 : 4;
    const bool chunked = din % chunk == 0 && dout % chunk == 0 && din >= 32 && dout >= 32 && B * T >= 16;
    if (!(dt == PEX_BF16 && bf16_supports(B, T, din, dout)) && din > 65535 * (int64_t)(dt == PEX_F32 && chunked ? 128 : 64)) return PEX_ERR_SHAPE;
    return PEX_OK;
}

static pex_status check_vec_args(const void* A, const void* C, int64_t B, int64_t T, int64_t d, pex_dtype dt, uint32_t want, float* s_id,
                                 float* s_sq, float* s_sign)
{
    if (!A) return PEX_ERR_NULL;
    if (want == 0 || (want & ~7u)) return PEX_ERR_PHI;
    float* outs[3] = {(want & PEX_WANT_IDENTITY) ? s_id : nullptr, (want & PEX_WANT_SQUARE) ? s_sq : nullptr,
                      (want & PEX_WANT_SIGN) ? s_sign : nullptr};
    for (int phi = 0; phi < 3; ++phi)
        if ((want & (1u << phi)) && !outs[phi]) return PEX_ERR_NULL;
    if (dt != PEX_F32 && dt != PEX_BF16) return PEX_ERR_DTYPE;
    const int64_t lim = (int64_t)1 << 31;
    if (B < 1 || T < 1 || d < 1 || B >= lim || T >= lim || d >= lim || B * T >= lim) return PEX_ERR_SHAPE;
    const uintptr_t esz = dt == PEX_BF16 ? 2 : 4;
    if (((uintptr_t)A | (uintptr_t)C) & (esz - 1)) return PEX_ERR_ALIGN;
    if (((uintptr_t)outs[0] | (uintptr_t)outs[1] | (uintptr_t)outs[2]) & 3u) return PEX_ERR_ALIGN;
    if (B * plan_vec_stat(B, T, d, dt).nrange >= 65536) return PEX_ERR_SHAPE;      // grid limit of the second launch dimension
    return PEX_OK;
}

// the partial sums of a plan without wide columns
static hipError_t reduce_whole(const ReduceOutputs& io, int count, const StatPlan& plan, hipStream_t stream)
{
    const int64_t n = plan.din * plan.dout;
    if (plan.dout == plan.out_cols) return launch_reduce_partials(io, count, plan.nsplit, n, 1, plan.out_rows * plan.out_cols, 0, 0, stream);
    return launch_reduce_partials(io, count, plan.nsplit, n, plan.out_rows, plan.out_cols, plan.dout, plan.out_cols, stream);
}

// The copies a plan asks for, at the front of the workspace; X and G are turned into what the kernels read.
static hipError_t make_copies(const StatPlan& plan, const void*& X, const void*& G, int64_t rows, void* workspace, bool made,
                              hipStream_t stream)
{
    if (plan.copy_bytes == 0) return hipSuccess;
    uint16_t* x = plan.copy_x ? (uint16_t*)workspace : nullptr;
    uint16_t* g = plan.copy_g ? (uint16_t*)workspace + (plan.copy_x ? rows * plan.din * (plan.square_halves ? 2 : 1) : 0) : nullptr;
    hipError_t e = hipSuccess;
    if (!made) {
        if (!plan.square_halves && plan.din == plan.out_rows && plan.dout == plan.out_cols) {       // squares of rows that are whole chunks
            e = launch_square_bf16(X, x, rows * plan.din, stream);
            if (e == hipSuccess) e = launch_square_bf16(G, g, rows * plan.dout, stream);
        } else e = launch_pad_rows(X, x, G, g, rows, plan.out_rows, plan.out_cols, plan.square_halves, stream);
    }
    if (x) X = x;
    if (g) G = g;
    return e;
}

static bool same_copies(const StatPlan& a, const StatPlan& b)
{
    return a.copy_bytes > 0 && a.copy_bytes == b.copy_bytes && a.copy_x == b.copy_x && a.copy_g == b.copy_g && a.din == b.din && a.dout == b.dout &&
           a.square_halves == b.square_halves;
}

// front: a plan whose copies the workspace already begins with
static pex_status run_stat(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt,
                           Mode mode, float* S, void* workspace, size_t workspace_bytes, hipStream_t stream,
                           const float* weight = nullptr, float alpha = 0.f, const StatPlan* front = nullptr)
{
    const StatPlan plan = plan_within(B, T, din, dout, dt, mode, workspace ? workspace_bytes : 0);
    float* out = S;
    if (plan.query_bytes > 0) {
        if (!workspace || workspace_bytes < plan.query_bytes) return PEX_ERR_WORKSPACE;
        if ((uintptr_t)workspace & 15u) return PEX_ERR_ALIGN;
    }
    float* partials = (float*)((char*)workspace + plan.copy_bytes);
    if (plan.nsplit > 1) out = partials;
    hipError_t e = make_copies(plan, X, G, B * T, workspace, front && same_copies(plan, *front), stream);
    if (e != hipSuccess) return PEX_ERR_HIP;
    din = plan.din;
    dout = plan.dout;
    if (plan.square_halves) {
        StatPlan part = plan;               // one of the four contractions: a result of the operands' widths
        part.out_rows = din;
        part.out_cols = dout;
        const int64_t n = din * dout, xhalf = B * T * din, ghalf = B * T * dout;
        for (int k = 0; k < 4 && e == hipSuccess; ++k) {
            float* dst = partials + (int64_t)k * plan.nsplit * n;
            e = launch_stat_bf16((const uint16_t*)X + (k / 2) * xhalf, (const uint16_t*)G + (k % 2) * ghalf, B, T, din, dout, MODE_IDENTITY, part, dst,
                                 dst, stream);
        }
        if (e == hipSuccess) e = launch_reduce_partials({{partials}, {S}}, 1, 4 * plan.nsplit, n, plan.out_rows, plan.out_cols, dout, plan.out_cols, stream,
                                       plan.nsplit);
        return e == hipSuccess ? PEX_OK : PEX_ERR_HIP;
    }
    if (plan.small_kw > 0) {
        e = launch_stat_small(X, G, B, T, din, dout, dt, mode, plan, out, stream, weight, nullptr, alpha);
    } else if (mode == MODE_TOKEN_SQ && plan.copy_bytes > 0) {
        e = launch_stat_bf16(X, G, B, T, din, dout, MODE_IDENTITY, plan, S, partials, stream);       // the copies hold the squares
    } else if (plan.kernel == 2) {
        e = launch_stat_f32(X, G, B, T, din, dout, mode, plan, out, stream, weight, nullptr, alpha);
    } else if (mode == MODE_POWER) {
        e = plan.kernel == 1 ? launch_power_bf16(X, G, alpha, B, T, din, dout, plan, S, partials, stream)
                             : launch_stat_generic(X, G, B, T, din, dout, dt, mode, plan, out, stream, nullptr, nullptr, alpha);
    } else if (mode == MODE_WEIGHTED) {
        e = plan.kernel == 1 ? launch_weighted_bf16(X, G, weight, B, T, din, dout, plan, S, partials, stream)
                             : launch_stat_generic(X, G, B, T, din, dout, dt, mode, plan, out, stream, weight, nullptr);
    } else if (plan.kernel == 1) e = launch_stat_bf16(X, G, B, T, din, dout, mode, plan, S, partials, stream);
    else e = launch_stat_generic(X, G, B, T, din, dout, dt, mode, plan, out, stream);
    if (e != hipSuccess) return PEX_ERR_HIP;
    // partial sums have the operands' widths, S the layer's own
    const int64_t rows = plan.out_rows, cols = plan.out_cols;
    if (plan.wide_cols > 0) {
        // the wide part's partial sums come first in the workspace, then those of the columns beyond it
        if (plan.wide_nsplit > 1) {
            const int64_t mine = plan.wide_cols < cols ? plan.wide_cols : cols;
            e = launch_reduce_partials({{partials}, {S}}, 1, plan.wide_nsplit, din * plan.wide_cols, rows, mine, plan.wide_cols, cols, stream);
            if (e != hipSuccess) return PEX_ERR_HIP;
        }
        const int64_t rest = dout - plan.wide_cols;
        if (plan.nsplit > 1 && rest > 0) {
            const float* rest_partials = (const float*)((const char*)partials + plan.wide_ws_bytes);
            e = launch_reduce_partials({{rest_partials}, {S + plan.wide_cols}}, 1, plan.nsplit, din * rest, rows, cols - plan.wide_cols, rest, cols,
                                       stream);
            if (e != hipSuccess) return PEX_ERR_HIP;
        }
    } else if (plan.nsplit > 1) {
        e = plan.sign_bytes ? launch_reduce_sign_bytes(partials, plan.nsplit, rows, cols, S, stream)
                            : reduce_whole({{partials}, {S}}, 1, plan, stream);
        if (e != hipSuccess) return PEX_ERR_HIP;
    }
    return PEX_OK;
}

// Identity and square of few long examples of a bf16 layer: M_b of every example by the kernel of plain contractions -- one register tile
// on 256 x 256 blocks, where both statistics beside it leave 256 x 128 -- into the workspace, and the sums over b, in the groups of `pair`
// and with the same bits, in a second pass.  A round of blocks takes 12 us (16 after another) and an example's multiply-adds, at 6.25e12 FLOP/s
// a compute unit on a full chip and up to 8.5 where few are busy (the eight-wave kernel, of examples below 1024 tokens, 7.6); the second pass 2.5 us
// and its bytes at 7 TB/s, or 0.6 us for every four examples where its few workgroups wait for their chains of loads (218 examples of 300 tokens,
// 208 x 416: 85 workgroups, 32 us for 75 MB); what the memory-side cache does not hold 0.2 us a MB.  Of 929 layers of 1 to 256 examples estimates
// within 10 % for four in five.  The pair's estimate is right where its blocks are one round, 5 % low for long examples, else 10 to 25 % low: so much more
// this may be.  687 of the layers are taken and 1.19 times faster in the mean, the least 0.97; of the others, 0.93 in the mean, three would gain more than
// 10 %, at most 16.  Together in one launch -> so, us: 4 x 8192 tokens, 4096 x 4096 992 -> 860; 16 x 4096, 768 x 3072 411 -> 313; 16 x 4092,
// 1024 x 1024 155 -> 121; 7 x 3000, 3000 x 1000 231 -> 151; 8 x 684, 1280 x 1152 39.6 -> 33.8; but 12 x 1500, 2048 x 2048 157 -> 176; 211 x 289,
// 528 x 152 47 -> 73; 25 x 1302, 576 x 384 36 -> 43; 23 x 969, 2688 x 1536 271 -> 297.
// Returns how much of the pair's time that is, 1 where it is not taken, beside estimates of many rounds of pairs (of 45 blocks of layers that change
// with it 44 are on the faster way, 30 if this is divided by what the layer's own estimate is low).
static double examples_share(int64_t B, int64_t T, int64_t din, int64_t dout, const StatPlan& pair)
{
    if (pair.kernel != 1 || pair.copy_bytes > 0 || T < 256) return 1.0;
    const double bytes = (double)din * (double)dout * 4.0, stored = (double)B * bytes;
    if (stored > 512.0 * 1048576.0) return 1.0;
    for (int k = 0; k < PLAN_OPTIONS; ++k)
        if (option(k) != DEFAULT_OPTIONS[k]) return 1.0;       // the options are about the other plans
    int bm, bn;
    bf16_tile_shape(MODE_IDENTITY, B, &bm, &bn);
    const int64_t wgs = ((din + bm - 1) / bm) * ((dout + bn - 1) / bn) * B, rounds = (wgs + 255) / 256;
    const double rate = T >= 1024 ? 8.5e12 - 2.25e12 * (double)wgs / (double)(256 * rounds) : 7.6e12;
    const double moved = (stored + 2.0 * bytes) / 7.0e12, chain = 0.6e-6 * (double)((B + 3) / 4);
    double t = (double)rounds * (16.0e-6 + 2.0 * (double)T * bm * bn / rate) - 4.0e-6 + 2.5e-6 + (moved > chain ? moved : chain);
    if (stored > 200.0e6) t += 0.2e-12 * (stored - 200.0e6);
    const bool several_rounds = bf16_pair_blocks(din, dout) * pair.nsplit > 256, long_ones = T >= 1536;
    const double most = several_rounds ? (long_ones ? 1.2 : 1.1) : (long_ones ? 1.05 : 1.0);
    return t < most * pair.seconds ? t / (1.25 * pair.seconds) : 1.0;
}

MultiPlan plan_multi(int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt, uint32_t want, bool allow_pad, bool allow_small, bool allow_examples)
{
    MultiPlan m{};
    const int n = __builtin_popcount(want);
    // (what shares a contraction of fp32 layers on the bf16 matrix cores is identity and square only)
    constexpr uint32_t BOTH = PEX_WANT_IDENTITY | PEX_WANT_SQUARE;
    // On the kernel of small layers any of them share one, with signs up to the number of tiles signs alone take it for.
    StatPlan sq = plan_stat(B, T, din, dout, dt, MODE_SQUARE, false, allow_pad, allow_small);
    const bool small = n >= 2 && sq.small_kw > 0 && (want == BOTH || small_tiles(din, dout) <= 256);
    if (!small) sq = plan_stat(B, T, din, dout, dt, MODE_SQUARE, false, allow_pad && (dt != PEX_F32 || want == BOTH), false);
    // Three wanted: all from one contraction while the sign counts fit bytes; otherwise identity and square share a
    // contraction and sign keeps its own.  On fp32 layers sign shares one only as bytes.
    m.pair_want = want;
    if (!small && sq.kernel == 1 && n == 3 && !bf16_triple_supported(sq)) m.pair_want = BOTH;
    if (!small && sq.kernel == 2 && !f32_bytes_suffice(sq)) m.pair_want = want & BOTH;
    m.pair = __builtin_popcount(m.pair_want) >= 2 && (sq.kernel != 0 || small);
    if (m.pair) {
        m.single_want = want & ~m.pair_want;
        m.pair_plan = sq;
        m.query_bytes = small ? __builtin_popcount(m.pair_want) * sq.ws_bytes : sq.copy_bytes + __builtin_popcount(m.pair_want) * (sq.query_bytes - sq.copy_bytes);
    } else {
        m.pair_want = 0;
        m.single_want = want;
    }
    if (allow_examples && stored_examples() && want == BOTH && m.pair && !small && examples_share(B, T, din, dout, sq) < 1.0) {
        m.examples = true;
        const size_t need = (size_t)B * (size_t)din * (size_t)dout * sizeof(float);
        if (need > m.query_bytes) m.query_bytes = need;
    }
    for (int phi = 0; phi < 3; ++phi)
        if (m.single_want & (1u << phi)) {
            const size_t w = plan_stat(B, T, din, dout, dt, (Mode)phi, true, allow_pad, allow_small).query_bytes;
            if (w > m.query_bytes) m.query_bytes = w;     // passes run one after the other on the stream and reuse it
        }
    if (small) {
        const size_t without = plan_multi(B, T, din, dout, dt, want, allow_pad, false, false).query_bytes;
        if (without > m.query_bytes) m.query_bytes = without;
    }
    return m;
}

// The plan of a call that has `bytes` of workspace at `workspace`, as plan_within; what a layer needs at least has no room for its M_b.
// (A layer that needs none runs beside a workspace at any address.)
MultiPlan plan_multi_within(int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt, uint32_t want, const void* workspace, size_t bytes)
{
    if (!workspace) bytes = 0;
    const MultiPlan first = plan_multi(B, T, din, dout, dt, want, true, true, ((uintptr_t)workspace & 15u) == 0);
    if (first.query_bytes <= bytes) return first;
    for (const bool allow_pad : {true, false}) {
        const MultiPlan m = plan_multi(B, T, din, dout, dt, want, allow_pad, false, false);
        if (m.query_bytes <= bytes) return m;
    }
    return first;
}

// ---- identity and square of several bf16 layers of one batch in one launch (pex_stat_pair_batch)

// A layer that may share it: by itself it would be one launch of 256 x 128 blocks on the operands as they are.
static bool pair_joins(int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt)
{
    if (dt != PEX_BF16) return false;
    for (int k = 0; k < PLAN_OPTIONS; ++k)
        if (option(k) != DEFAULT_OPTIONS[k]) return false;       // the options are about the plans of single layers
    const StatPlan p = plan_stat(B, T, din, dout, dt, MODE_SQUARE, false, true, false);
    return p.kernel == 1 && p.copy_bytes == 0 && din % 8 == 0 && dout % 8 == 0;
}

struct PairBatchPlan {
    bool joint;
    int64_t nsplit, per;      // groups of examples of every layer
    size_t ws_bytes;
};

// The layers' blocks as those of one layer, all cut into the same number of groups, against each by itself, whichever kernel that takes; an example counted with its
// fold, 3 us for the start and end of a workgroup, 5 for a launch, partial sums as for single layers.  (Numbers of their own, so that shorter
// groups fill the last round, were estimated over the layers of transformer blocks: none to 3 % better, 8 in one of six.)
// A sum is rounded once per example of a group and once per group, beside what the sums over the tokens leave: 34 blocks' errors against
// 64-bit sums are, in 1e-16 of the 2-norm squared, 10 T/32 + 3.5 (examples of a group + groups) of S_id, (0.5 + 81/B) T/32 + 1.9 (..) of S_sq, within
// 2 and 5 %.  The groups are such that neither grows by more than 2.5 % over any layer by itself on these blocks.  (Bounded by the layer that
// is rounded most often, B=22, T=70, d=768: the whole step 374 us instead of 461, but S_id of the projection 7.8e-8 off instead of 5.5e-8.)
static PairBatchPlan make_pair_batch_plan(int64_t B, int64_t T, int count, const int64_t* din, const int64_t* dout, bool stored)
{
    constexpr double START = 3.0e-6, LAUNCH = 5.0e-6, RATE = 4.0e12, TAKEN = 0.8;      // (that part of such an estimate, see make_plan)
    const double unit = bf16_unit_with_fold(MODE_SQUARE, true, T, 256, 128);
    auto seconds = [&](int64_t blocks, int64_t ns, int64_t per, double bytes) {
        const double t = (double)((blocks * ns + 255) / 256) * ((double)per * unit + START);
        return ns > 1 ? t + (double)(2 * ns + 1) * bytes / RATE : t;
    };
    const double slabs = (double)T / 32.0, of_square = (0.25 + 43.0 / (double)B) * slabs, of_tokens = 2.9 * slabs < of_square ? 2.9 * slabs : of_square;
    int64_t blocks = 0, fewest_roundings = INT64_MAX;
    double bytes = 0.0, alone = 0.0;
    for (int k = 0; k < count; ++k) {
        const int64_t own = bf16_pair_blocks(din[k], dout[k]);
        const double own_bytes = 2.0 * (double)din[k] * (double)dout[k] * sizeof(float);
        const StatPlan p = plan_stat(B, T, din[k], dout[k], PEX_BF16, MODE_SQUARE, false, true, false), by_itself = plan_stat(B, T, din[k], dout[k], PEX_BF16, MODE_SQUARE, false);
        alone += by_itself.small_kw > 0 ? by_itself.seconds
                                        : TAKEN * (stored ? examples_share(B, T, din[k], dout[k], p) : 1.0) * (seconds(own, p.nsplit, p.per_split, own_bytes) + (p.nsplit > 1 ? 2.0 : 1.0) * LAUNCH);
        blocks += own;
        bytes += own_bytes;
        if (p.per_split + p.nsplit < fewest_roundings) fewest_roundings = p.per_split + p.nsplit;
    }
    PairBatchPlan plan{};
    if (count < 2 || blocks >= ((int64_t)1 << 20)) return plan;
    double best = alone;
    const int64_t most = B < 32 ? B : 32;
    for (int64_t ns = 1; ns <= most; ns = more_groups(B, ns)) {
        const int64_t per = (B + ns - 1) / ns, groups = (B + per - 1) / per;
        const double cost = TAKEN * (seconds(blocks, groups, per, bytes) + (groups > 1 ? 2.0 : 1.0) * LAUNCH);
        if (cost >= best || of_tokens + (double)(per + groups) > 1.05 * (of_tokens + (double)fewest_roundings) || (groups > 1 && (double)groups * bytes > 512.0 * 1048576.0)) continue;
        best = cost;
        plan = PairBatchPlan{true, groups, per, groups > 1 ? (size_t)groups * (size_t)bytes : 0};
    }
    return plan;
}

// Kept like the plans of plan_stat, eight a thread.
static PairBatchPlan plan_pair_batch(int64_t B, int64_t T, int count, const int64_t* din, const int64_t* dout, bool stored)
{
    struct Kept {
        int64_t key[4 + 2 * PAIR_BATCH];
        PairBatchPlan plan;
        bool valid;
    };
    static thread_local Kept kept[8];
    int64_t key[4 + 2 * PAIR_BATCH] = {B, T, count, stored};
    uint64_t h = 0;
    for (int k = 0; k < count; ++k) {
        key[4 + 2 * k] = din[k];
        key[5 + 2 * k] = dout[k];
    }
    for (const int64_t x : key) h = (h ^ (uint64_t)x) * 0x9e3779b97f4a7c15ull;
    Kept& at = kept[h >> 61];
    bool same = at.valid;
    for (int k = 0; k < 4 + 2 * PAIR_BATCH; ++k) same = same && key[k] == at.key[k];
    if (same) return at.plan;
    at.plan = make_pair_batch_plan(B, T, count, din, dout, stored);
    for (int k = 0; k < 4 + 2 * PAIR_BATCH; ++k) at.key[k] = key[k];
    at.valid = true;
    return at.plan;
}

// The items from `from` on that go together: how many items this step covers, and the plan if they share a launch.  stored = false: against each
// by itself without its M_b in the workspace.
static int next_pair_group(const pex_pair_item* items, int32_t count, int32_t from, int64_t B, int64_t T, pex_dtype dt, bool stored, PairBatchPlan* plan)
{
    int64_t din[PAIR_BATCH], dout[PAIR_BATCH];
    int n = 0;
    while (from + n < count && n < PAIR_BATCH && pair_joins(B, T, items[from + n].din, items[from + n].dout, dt)) {
        din[n] = items[from + n].din;
        dout[n] = items[from + n].dout;
        ++n;
    }
    *plan = PairBatchPlan{};
    if (n >= 2) *plan = plan_pair_batch(B, T, n, din, dout, stored);
    return n > 0 ? n : 1;
}

}  // namespace pex

using namespace pex;

extern "C" {

const char* pex_status_string(pex_status s)
{
    switch (s) {
    case PEX_OK: return "PEX_OK";
    case PEX_ERR_NULL: return "PEX_ERR_NULL: a required pointer is NULL";
    case PEX_ERR_SHAPE: return "PEX_ERR_SHAPE: a dimension is out of range";
    case PEX_ERR_DTYPE: return "PEX_ERR_DTYPE: unknown storage type";
    case PEX_ERR_PHI: return "PEX_ERR_PHI: unknown phi or optimizer variant";
    case PEX_ERR_ALIGN: return "PEX_ERR_ALIGN: a pointer is not 16-byte aligned";
    case PEX_ERR_WORKSPACE: return "PEX_ERR_WORKSPACE: workspace missing or too small";
    case PEX_ERR_HIP: return "PEX_ERR_HIP: the HIP runtime reported an error";
    case PEX_ERR_TOO_LARGE: return "PEX_ERR_TOO_LARGE: the call needs more scratch than the library's static buffer holds";
    }
    return "PEX: unknown status";
}

int pex_version(void) { return PEX_VERSION; }

pex_status pex_set_option(pex_option opt, int32_t value)
{
    if (!known_option(opt)) return PEX_ERR_PHI;
    if (value != clamp_option(opt, value)) return PEX_ERR_SHAPE;
    options().v[opt].store(value);
    return PEX_OK;
}

int32_t pex_get_option(pex_option opt)
{
    if (!known_option(opt)) return -1;
    return option(opt);
}

size_t pex_stat_workspace_bytes(int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt, pex_phi phi)
{
    if (B < 1 || T < 1 || din < 1 || dout < 1) return 0;
    if (dt != PEX_F32 && dt != PEX_BF16) return 0;
    if (phi != PEX_PHI_IDENTITY && phi != PEX_PHI_SQUARE && phi != PEX_PHI_SIGN) return 0;
    return plan_stat(B, T, din, dout, dt, (Mode)phi).query_bytes;
}

pex_status pex_stat(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt,
                    pex_phi phi, float* S, void* workspace, size_t workspace_bytes, pex_stream_t stream)
{
    const pex_status st = check_stat_args(X, G, B, T, din, dout, dt, S);
    if (st != PEX_OK) return st;
    if (phi != PEX_PHI_IDENTITY && phi != PEX_PHI_SQUARE && phi != PEX_PHI_SIGN) return PEX_ERR_PHI;
    return run_stat(X, G, B, T, din, dout, dt, (Mode)phi, S, workspace, workspace_bytes, (hipStream_t)stream);
}

pex_status pex_stat_noalloc(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt,
                            pex_phi phi, float* S, pex_stream_t stream)
{
    const pex_status st = check_stat_args(X, G, B, T, din, dout, dt, S);
    if (st != PEX_OK) return st;
    if (phi != PEX_PHI_IDENTITY && phi != PEX_PHI_SQUARE && phi != PEX_PHI_SIGN) return PEX_ERR_PHI;
    const size_t limit = (size_t)PEX_NOALLOC_SCRATCH_BYTES;
    const size_t need = plan_within(B, T, din, dout, dt, (Mode)phi, limit).query_bytes;
    if (need > limit) return PEX_ERR_TOO_LARGE;
    void* ws = nullptr;
    if (need > 0 && scratch_address(&ws) != hipSuccess) return PEX_ERR_HIP;
    // Every partial sum the reduction reads is written by the contraction of the same call, so nothing in the
    // scratch has to start at zero.
    return run_stat(X, G, B, T, din, dout, dt, (Mode)phi, S, ws, limit, (hipStream_t)stream);
}

size_t pex_stat_multi_workspace_bytes(int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt, uint32_t want)
{
    if (B < 1 || T < 1 || din < 1 || dout < 1) return 0;
    if (dt != PEX_F32 && dt != PEX_BF16) return 0;
    if (want == 0 || (want & ~7u)) return 0;
    return plan_multi(B, T, din, dout, dt, want).query_bytes;
}

pex_status pex_stat_multi(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt,
                          uint32_t want, float* S_id, float* S_sq, float* S_sign, void* workspace,
                          size_t workspace_bytes, pex_stream_t stream)
{
    if (want == 0 || (want & ~7u)) return PEX_ERR_PHI;
    float* outs[3] = {(want & PEX_WANT_IDENTITY) ? S_id : nullptr, (want & PEX_WANT_SQUARE) ? S_sq : nullptr,
                      (want & PEX_WANT_SIGN) ? S_sign : nullptr};
    for (int phi = 0; phi < 3; ++phi) {
        if (!(want & (1u << phi))) continue;
        const pex_status st = check_stat_args(X, G, B, T, din, dout, dt, outs[phi]);
        if (st != PEX_OK) return st;
    }
    const size_t given = workspace ? workspace_bytes : 0;
    const MultiPlan m = plan_multi_within(B, T, din, dout, dt, want, workspace, workspace_bytes);
    if (m.query_bytes > 0) {
        if (!workspace || workspace_bytes < m.query_bytes) return PEX_ERR_WORKSPACE;
        if ((uintptr_t)workspace & 15u) return PEX_ERR_ALIGN;
    }
    hipStream_t hs = (hipStream_t)stream;
    StatPlan front{};       // whose copies the workspace begins with
    if (m.examples) {
        StatPlan each = m.pair_plan;       // one example a group
        each.nsplit = (int)B;
        each.per_split = T;
        float* M = (float*)workspace;
        if (launch_stat_bf16(X, G, B, T, din, dout, MODE_IDENTITY, each, M, M, hs) != hipSuccess) return PEX_ERR_HIP;
        return launch_fold_examples(M, B, m.pair_plan.per_split, din * dout, outs[0], outs[1], hs) == hipSuccess ? PEX_OK : PEX_ERR_HIP;
    }
    if (m.pair) {
        const StatPlan& p = front = m.pair_plan;
        const int64_t n = p.din * p.dout;
        const void *x = X, *g = G;
        if (make_copies(p, x, g, B * T, workspace, false, hs) != hipSuccess) return PEX_ERR_HIP;
        float* partials = (float*)((char*)workspace + p.copy_bytes);
        float* po[3] = {nullptr, nullptr, nullptr};
        int k = 0;
        for (int phi = 0; phi < 3; ++phi)
            if (m.pair_want & (1u << phi)) po[phi] = p.nsplit > 1 ? partials + (int64_t)(k++) * p.nsplit * n : outs[phi];
        const hipError_t e = p.small_kw > 0 ? launch_stat_small_multi(x, g, B, T, p.din, p.dout, dt, p, po[0], po[1], po[2], hs)
                             : p.kernel == 2 ? launch_stat_f32_multi(x, g, B, T, p.din, p.dout, p, po[0], po[1], po[2], hs)
                             : (__builtin_popcount(m.pair_want) == 3)
                                 ? launch_stat_bf16_triple(x, g, B, T, p.din, p.dout, p, po[0], po[1], po[2], hs)
                                 : launch_stat_bf16_pair(x, g, B, T, p.din, p.dout, p, po[0], po[1], po[2], hs);
        if (e != hipSuccess) return PEX_ERR_HIP;
        if (p.nsplit > 1) {
            ReduceOutputs io{};
            int count = 0;
            for (int phi = 0; phi < 3; ++phi)
                if (po[phi]) { io.partial[count] = po[phi]; io.S[count++] = outs[phi]; }
            if (reduce_whole(io, count, p, hs) != hipSuccess) return PEX_ERR_HIP;
        }
    }
    for (int phi = 0; phi < 3; ++phi) {
        if (!(m.single_want & (1u << phi))) continue;
        // what runs alone beside a shared contraction finds the padded copies made, if it reads the same ones
        const pex_status st = run_stat(X, G, B, T, din, dout, dt, (Mode)phi, outs[phi], workspace, workspace_bytes, hs, nullptr, 0.f, &front);
        front = plan_within(B, T, din, dout, dt, (Mode)phi, given);
        if (st != PEX_OK) return st;
    }
    return PEX_OK;
}

size_t pex_vec_stat_workspace_bytes(int64_t B, int64_t T, int64_t d, pex_dtype dt)
{
    if (B < 1 || T < 1 || d < 1) return 0;
    if (dt != PEX_F32 && dt != PEX_BF16) return 0;
    return plan_vec_stat(B, T, d, dt).ws_bytes;
}

pex_status pex_vec_stat(const void* A, const void* C, int64_t B, int64_t T, int64_t d, pex_dtype dt, uint32_t want,
                        float* s_id, float* s_sq, float* s_sign, void* workspace, size_t workspace_bytes,
                        pex_stream_t stream)
{
    const pex_status st = check_vec_args(A, C, B, T, d, dt, want, s_id, s_sq, s_sign);
    if (st != PEX_OK) return st;
    float* outs[3] = {(want & PEX_WANT_IDENTITY) ? s_id : nullptr, (want & PEX_WANT_SQUARE) ? s_sq : nullptr,
                      (want & PEX_WANT_SIGN) ? s_sign : nullptr};
    const VecPlan plan = plan_vec_stat(B, T, d, dt);
    if (!workspace || workspace_bytes < plan.ws_bytes) return PEX_ERR_WORKSPACE;
    if ((uintptr_t)workspace & 15u) return PEX_ERR_ALIGN;
    return launch_vec_stat(A, C, B, T, d, dt, plan, (float*)workspace, outs[0], outs[1], outs[2], (hipStream_t)stream) ==
                   hipSuccess
               ? PEX_OK
               : PEX_ERR_HIP;
}

size_t pex_stat_pair_batch_workspace_bytes(const pex_pair_item* items, int32_t count, int64_t B, int64_t T, pex_dtype dt)
{
    if (!items || count < 1 || B < 1 || T < 1 || (dt != PEX_F32 && dt != PEX_BF16)) return 0;
    for (int k = 0; k < count; ++k)
        if (items[k].din < 1 || items[k].dout < 1) return 0;
    size_t need = 0;
    PairBatchPlan plan;
    for (int k = 0; k < count;) {
        const int end = k + next_pair_group(items, count, k, B, T, dt, stored_examples(), &plan);
        if (plan.ws_bytes > need) need = plan.ws_bytes;
        for (; k < end; ++k) {
            // what each would need by itself, and room for its M_b only where it goes by itself
            const size_t own = plan_multi(B, T, items[k].din, items[k].dout, dt, PEX_WANT_IDENTITY | PEX_WANT_SQUARE, true, true, !plan.joint).query_bytes;
            if (own > need) need = own;
        }
    }
    return need;
}

pex_status pex_stat_pair_batch(const pex_pair_item* items, int32_t count, int64_t B, int64_t T, pex_dtype dt, void* workspace, size_t workspace_bytes,
                               pex_stream_t stream)
{
    if (!items) return PEX_ERR_NULL;
    if (count < 1) return PEX_ERR_SHAPE;
    constexpr uint32_t BOTH = PEX_WANT_IDENTITY | PEX_WANT_SQUARE;
    const size_t given = workspace ? workspace_bytes : 0;
    bool uses_workspace = false;
    for (int k = 0; k < count; ++k) {
        const pex_pair_item& it = items[k];
        for (const float* S : {it.S_id, it.S_sq}) {
            const pex_status st = check_stat_args(it.X, it.G, B, T, it.din, it.dout, dt, S);
            if (st != PEX_OK) return st;
        }
        const size_t need = plan_multi_within(B, T, it.din, it.dout, dt, BOTH, workspace, workspace_bytes).query_bytes;
        if (need > given) return PEX_ERR_WORKSPACE;
        uses_workspace = uses_workspace || need > 0;
    }
    if (uses_workspace && ((uintptr_t)workspace & 15u)) return PEX_ERR_ALIGN;
    hipStream_t hs = (hipStream_t)stream;
    for (int k = 0; k < count;) {
        PairBatchPlan plan;
        const int n = next_pair_group(items, count, k, B, T, dt, stored_examples(), &plan);
        if (n >= 2 && !plan.joint) {
            // each by itself only with the room that counts on
            bool room = true;
            for (int o = k; o < k + n; ++o) room = room && (plan_multi(B, T, items[o].din, items[o].dout, dt, BOTH).query_bytes <= given);
            if (!room || ((uintptr_t)workspace & 15u)) next_pair_group(items, count, k, B, T, dt, false, &plan);
        }
        if (!plan.joint || plan.ws_bytes > given || (plan.ws_bytes > 0 && ((uintptr_t)workspace & 15u))) {
            for (const int end = k + n; k < end; ++k) {
                const pex_pair_item& it = items[k];
                const pex_status st = pex_stat_multi(it.X, it.G, B, T, it.din, it.dout, dt, BOTH, it.S_id, it.S_sq, nullptr, workspace, workspace_bytes, stream);
                if (st != PEX_OK) return st;
            }
            continue;
        }
        PairItem layers[PAIR_BATCH];
        ReduceBatch sums{};
        float* partial = (float*)workspace;
        for (int o = 0; o < n; ++o) {
            const pex_pair_item& it = items[k + o];
            PairItem& l = layers[o] = PairItem{it.X, it.G, it.S_id, it.S_sq, it.din, it.dout};
            if (plan.nsplit == 1) continue;
            for (float** out : {&l.out_id, &l.out_sq}) {
                const int r = sums.count++;
                sums.S[r] = *out;
                sums.partial[r] = *out = partial;
                sums.n[r] = it.din * it.dout;
                partial += plan.nsplit * sums.n[r];
            }
        }
        if (launch_stat_bf16_pair_batch(layers, n, B, T, plan.nsplit, plan.per, hs) != hipSuccess) return PEX_ERR_HIP;
        if (sums.count > 0 && launch_reduce_batch(sums, (int)plan.nsplit, hs) != hipSuccess) return PEX_ERR_HIP;
        k += n;
    }
    return PEX_OK;
}

size_t pex_vec_stat_batch_workspace_bytes(const pex_vec_item* items, int32_t count, int64_t B, int64_t T, pex_dtype dt)
{
    if (!items || count < 1 || B < 1 || T < 1 || (dt != PEX_F32 && dt != PEX_BF16)) return 0;
    size_t total = 0;
    for (int k = 0; k < count; ++k) {
        if (items[k].d < 1) return 0;
        total += vec_batch_bytes(plan_vec_stat(B, T, items[k].d, dt));
    }
    return total;
}

pex_status pex_vec_stat_batch(const pex_vec_item* items, int32_t count, int64_t B, int64_t T, pex_dtype dt, uint32_t want, void* workspace,
                              size_t workspace_bytes, pex_stream_t stream)
{
    if (!items) return PEX_ERR_NULL;
    if (count < 1) return PEX_ERR_SHAPE;
    for (int k = 0; k < count; ++k) {
        const pex_vec_item& it = items[k];
        const pex_status st = check_vec_args(it.A, it.C, B, T, it.d, dt, want, it.s_id, it.s_sq, it.s_sign);
        if (st != PEX_OK) return st;
        if (!workspace || workspace_bytes < vec_batch_bytes(plan_vec_stat(B, T, it.d, dt))) return PEX_ERR_WORKSPACE;
    }
    if ((uintptr_t)workspace & 15u) return PEX_ERR_ALIGN;
    for (int k = 0; k < count;) {
        pex_vec_item group[VEC_BATCH];
        int n = 0;
        size_t bytes = 0;
        int64_t blocks = 0;
        for (; k < count && n < VEC_BATCH; ++k) {
            pex_vec_item it = items[k];
            const VecPlan plan = plan_vec_stat(B, T, it.d, dt);
            const int64_t own = (it.d + 63) / 64 * B * plan.nrange;       // at most: a launch holds fewer than 2^32 threads
            if (n > 0 && (bytes + vec_batch_bytes(plan) > workspace_bytes || blocks + own >= ((int64_t)1 << 23))) break;
            bytes += vec_batch_bytes(plan);
            blocks += own;
            if (!(want & PEX_WANT_IDENTITY)) it.s_id = nullptr;
            if (!(want & PEX_WANT_SQUARE)) it.s_sq = nullptr;
            if (!(want & PEX_WANT_SIGN)) it.s_sign = nullptr;
            group[n++] = it;
        }
        hipError_t e;
        if (n == 1) {       // alone: as pex_vec_stat, whose grid has two dimensions
            const pex_vec_item& it = group[0];
            e = launch_vec_stat(it.A, it.C, B, T, it.d, dt, plan_vec_stat(B, T, it.d, dt), (float*)workspace, it.s_id, it.s_sq, it.s_sign, (hipStream_t)stream);
        } else e = launch_vec_stat_batch(group, n, B, T, dt, workspace, (hipStream_t)stream);
        if (e != hipSuccess) return PEX_ERR_HIP;
    }
    return PEX_OK;
}

size_t pex_example_norms_workspace_bytes(int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt)
{
    if (B < 1 || T < 1 || din < 1 || dout < 1) return 0;
    if (dt != PEX_F32 && dt != PEX_BF16) return 0;
    return plan_stat(B, T, din, dout, dt, MODE_NORMS).query_bytes;
}

pex_status pex_example_norms(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt,
                             float* N, void* workspace, size_t workspace_bytes, pex_stream_t stream)
{
    pex_status st = check_stat_args(X, G, B, T, din, dout, dt, (const float*)0x10);
    if (st != PEX_OK) return st;
    if (!N) return PEX_ERR_NULL;
    if ((uintptr_t)N & 3u) return PEX_ERR_ALIGN;
    const StatPlan plan = plan_within(B, T, din, dout, dt, MODE_NORMS, workspace ? workspace_bytes : 0);
    if (!workspace || workspace_bytes < plan.query_bytes) return PEX_ERR_WORKSPACE;
    if ((uintptr_t)workspace & 15u) return PEX_ERR_ALIGN;
    hipStream_t hs = (hipStream_t)stream;
    char* front = (char*)workspace + plan.copy_bytes;
    float* partial = (float*)front;
    if (make_copies(plan, X, G, B * T, workspace, false, hs) != hipSuccess) return PEX_ERR_HIP;
    const int64_t kin = plan.din, kout = plan.dout;
    hipError_t e;
    int64_t nparts;
    if (plan.small_kw > 0) {
        nparts = small_tiles(kin, kout) * plan.small_kw;
        e = launch_stat_small(X, G, B, T, kin, kout, dt, MODE_NORMS, plan, nullptr, hs, nullptr, partial);
    } else if (plan.gram_wide) {
        nparts = gram_wide_partials(T);
        void* park = front + (((size_t)nparts * (size_t)B * sizeof(float) + 255) & ~(size_t)255);
        e = launch_gram_wide(X, G, B, T, kin, kout, partial, park, hs);
    } else if (plan.gram) {
        nparts = gram_norm_partials(T);
        e = launch_gram_norms(X, G, B, T, kin, kout, partial, hs);
    } else if (plan.kernel == 1) {
        nparts = bf16_norm_partials(kin, kout);
        e = launch_norms_bf16(X, G, B, T, kin, kout, plan, partial, hs);
    } else if (plan.kernel == 2) {
        nparts = plan.f32_split ? 4 * f32_split_blocks(kin, kout) : f32_norm_partials(kin, kout);
        e = launch_stat_f32(X, G, B, T, kin, kout, MODE_NORMS, plan, nullptr, hs, nullptr, partial);
    } else {
        nparts = generic_norm_partials(kin, kout);
        e = launch_stat_generic(X, G, B, T, kin, kout, dt, MODE_NORMS, plan, nullptr, hs, nullptr, partial);
    }
    if (e != hipSuccess) return PEX_ERR_HIP;
    return launch_reduce_norms(partial, nparts, B, N, hs) == hipSuccess ? PEX_OK : PEX_ERR_HIP;
}

size_t pex_weighted_sum_workspace_bytes(int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt)
{
    if (B < 1 || T < 1 || din < 1 || dout < 1) return 0;
    if (dt != PEX_F32 && dt != PEX_BF16) return 0;
    return plan_stat(B, T, din, dout, dt, MODE_WEIGHTED).query_bytes;
}

pex_status pex_weighted_sum(const void* X, const void* G, const float* w, int64_t B, int64_t T, int64_t din, int64_t dout,
                            pex_dtype dt, float* S, void* workspace, size_t workspace_bytes, pex_stream_t stream)
{
    const pex_status st = check_stat_args(X, G, B, T, din, dout, dt, S);
    if (st != PEX_OK) return st;
    if (!w) return PEX_ERR_NULL;
    if ((uintptr_t)w & 3u) return PEX_ERR_ALIGN;
    return run_stat(X, G, B, T, din, dout, dt, MODE_WEIGHTED, S, workspace, workspace_bytes, (hipStream_t)stream, w);
}

pex_status pex_clip_weights(const float* N, int64_t B, int32_t nlayers, float max_norm, float* w, pex_stream_t stream)
{
    if (!N || !w) return PEX_ERR_NULL;
    if (B < 1 || nlayers < 1 || B >= ((int64_t)1 << 31) || !(max_norm > 0.f)) return PEX_ERR_SHAPE;
    if (((uintptr_t)N | (uintptr_t)w) & 3u) return PEX_ERR_ALIGN;
    return launch_clip_weights(N, B, nlayers, max_norm, w, (hipStream_t)stream) == hipSuccess ? PEX_OK : PEX_ERR_HIP;
}

size_t pex_stat_power_workspace_bytes(int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt)
{
    if (B < 1 || T < 1 || din < 1 || dout < 1) return 0;
    if (dt != PEX_F32 && dt != PEX_BF16) return 0;
    return plan_stat(B, T, din, dout, dt, MODE_POWER).query_bytes;
}

pex_status pex_stat_power(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt,
                          float alpha, float* S, void* workspace, size_t workspace_bytes, pex_stream_t stream)
{
    const pex_status st = check_stat_args(X, G, B, T, din, dout, dt, S);
    if (st != PEX_OK) return st;
    if (!(alpha > 0.f) || !(alpha <= 64.f)) return PEX_ERR_PHI;
    return run_stat(X, G, B, T, din, dout, dt, MODE_POWER, S, workspace, workspace_bytes, (hipStream_t)stream, nullptr, alpha);
}

pex_status pex_token_norms(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt,
                           float* N_tok, pex_stream_t stream)
{
    const pex_status st = check_stat_args(X, G, B, T, din, dout, dt, (const float*)0x10);
    if (st != PEX_OK) return st;
    if (!N_tok) return PEX_ERR_NULL;
    if ((uintptr_t)N_tok & 3u) return PEX_ERR_ALIGN;
    return launch_token_norms(X, G, B * T, din, dout, dt, N_tok, (hipStream_t)stream) == hipSuccess ? PEX_OK : PEX_ERR_HIP;
}

size_t pex_token_sq_workspace_bytes(int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt)
{
    if (B < 1 || T < 1 || din < 1 || dout < 1) return 0;
    if (dt != PEX_F32 && dt != PEX_BF16) return 0;
    return plan_stat(B, T, din, dout, dt, MODE_TOKEN_SQ).query_bytes;
}

pex_status pex_token_sq(const void* X, const void* G, int64_t B, int64_t T, int64_t din, int64_t dout, pex_dtype dt,
                        float* S_tok, void* workspace, size_t workspace_bytes, pex_stream_t stream)
{
    const pex_status st = check_stat_args(X, G, B, T, din, dout, dt, S_tok);
    if (st != PEX_OK) return st;
    return run_stat(X, G, B, T, din, dout, dt, MODE_TOKEN_SQ, S_tok, workspace, workspace_bytes, (hipStream_t)stream);
}

pex_status pex_adam_update(float* theta, float* m, float* v, const float* S_id, const float* S_sq, int64_t n,
                           pex_adam_variant variant, const pex_adam_params* p, pex_stream_t stream)
{
    if (!theta || !m || !v || !S_id || !p) return PEX_ERR_NULL;
    if (variant != PEX_ADAM && variant != PEX_MICROADAM && variant != PEX_MICROADAM_VAR && variant != PEX_MICROADAM_MSQ)
        return PEX_ERR_PHI;
    if (variant != PEX_ADAM && !S_sq) return PEX_ERR_NULL;
    if (n < 1 || p->step < 1 || p->B < 1) return PEX_ERR_SHAPE;
    if ((variant == PEX_MICROADAM_VAR || variant == PEX_MICROADAM_MSQ) && p->B < 2) return PEX_ERR_SHAPE;
    if (((uintptr_t)theta | (uintptr_t)m | (uintptr_t)v | (uintptr_t)S_id | (uintptr_t)S_sq) & 15u) return PEX_ERR_ALIGN;
    return launch_adam_update(theta, m, v, S_id, S_sq, n, variant, *p, (hipStream_t)stream) == hipSuccess ? PEX_OK
                                                                                                           : PEX_ERR_HIP;
}

size_t pex_embed_stat_workspace_bytes(int64_t B, int64_t T, int64_t V, int64_t d)
{
    const int64_t lim = (int64_t)1 << 31;
    if (B < 1 || T < 1 || V < 1 || d < 1 || B >= lim || T >= lim || B * T >= lim || V >= lim - 1) return 0;
    return embed_workspace(B, T, V, d);
}

pex_status pex_embed_stat(const void* ids, int32_t ids_bytes, const void* G, int64_t B, int64_t T, int64_t V, int64_t d,
                          pex_dtype dt, uint32_t want, float* S_id, float* S_sq, float* S_sign, void* workspace,
                          size_t workspace_bytes, pex_stream_t stream)
{
    if (want == 0 || (want & ~7u)) return PEX_ERR_PHI;
    if (!ids || !G) return PEX_ERR_NULL;
    if ((want & PEX_WANT_IDENTITY) && !S_id) return PEX_ERR_NULL;
    if ((want & PEX_WANT_SQUARE) && !S_sq) return PEX_ERR_NULL;
    if ((want & PEX_WANT_SIGN) && !S_sign) return PEX_ERR_NULL;
    if (dt != PEX_F32 && dt != PEX_BF16) return PEX_ERR_DTYPE;
    if (ids_bytes != 4 && ids_bytes != 8) return PEX_ERR_DTYPE;
    const int64_t lim = (int64_t)1 << 31;
    if (B < 1 || T < 1 || V < 1 || d < 1 || B >= lim || T >= lim || B * T >= lim || V >= lim - 1 || d >= lim) return PEX_ERR_SHAPE;
    uintptr_t al = (uintptr_t)G;
    if (want & PEX_WANT_IDENTITY) al |= (uintptr_t)S_id;
    if (want & PEX_WANT_SQUARE) al |= (uintptr_t)S_sq;
    if (want & PEX_WANT_SIGN) al |= (uintptr_t)S_sign;
    if ((al & 15u) || ((uintptr_t)ids & (uintptr_t)(ids_bytes - 1))) return PEX_ERR_ALIGN;
    if (!workspace || workspace_bytes < embed_workspace_least(B, T, V, d)) return PEX_ERR_WORKSPACE;
    if ((uintptr_t)workspace & 15u) return PEX_ERR_ALIGN;
    return launch_embed_stat(ids, ids_bytes, G, B, T, V, d, dt, want, S_id, S_sq, S_sign, workspace, workspace_bytes,
                             (hipStream_t)stream) == hipSuccess
               ? PEX_OK
               : PEX_ERR_HIP;
}

size_t pex_sum_squares_workspace_bytes(int64_t n) { return n < 1 ? 0 : sum_squares_workspace(n); }

pex_status pex_sum_squares(const float* x, int64_t n, double* acc, int32_t accumulate, void* workspace, size_t workspace_bytes,
                           pex_stream_t stream)
{
    if (!x || !acc) return PEX_ERR_NULL;
    if (n < 1) return PEX_ERR_SHAPE;
    if (((uintptr_t)x & 15u) || ((uintptr_t)acc & 7u)) return PEX_ERR_ALIGN;
    if (!workspace || workspace_bytes < sum_squares_workspace(n)) return PEX_ERR_WORKSPACE;
    if ((uintptr_t)workspace & 15u) return PEX_ERR_ALIGN;
    return launch_sum_squares(x, n, acc, accumulate, (double*)workspace, (hipStream_t)stream) == hipSuccess ? PEX_OK : PEX_ERR_HIP;
}

pex_status pex_adam_update_clipped(float* theta, float* m, float* v, const float* S_id, const float* S_sq, int64_t n,
                                   pex_adam_variant variant, const pex_adam_params* p, const double* sum_sq, float max_norm,
                                   pex_stream_t stream)
{
    if (!theta || !m || !v || !S_id || !p || !sum_sq) return PEX_ERR_NULL;
    if (variant != PEX_ADAM && variant != PEX_MICROADAM && variant != PEX_MICROADAM_VAR && variant != PEX_MICROADAM_MSQ)
        return PEX_ERR_PHI;
    if (variant != PEX_ADAM && !S_sq) return PEX_ERR_NULL;
    if (n < 1 || p->step < 1 || p->B < 1 || !(max_norm > 0.f)) return PEX_ERR_SHAPE;
    if ((variant == PEX_MICROADAM_VAR || variant == PEX_MICROADAM_MSQ) && p->B < 2) return PEX_ERR_SHAPE;
    if (((uintptr_t)theta | (uintptr_t)m | (uintptr_t)v | (uintptr_t)S_id | (uintptr_t)S_sq) & 15u) return PEX_ERR_ALIGN;
    if ((uintptr_t)sum_sq & 7u) return PEX_ERR_ALIGN;
    return launch_adam_update(theta, m, v, S_id, S_sq, n, variant, *p, (hipStream_t)stream, sum_sq, max_norm) == hipSuccess
               ? PEX_OK
               : PEX_ERR_HIP;
}

size_t pex_adam_step_workspace_bytes(const pex_step_tensor* tensors, int32_t count)
{
    if (!tensors || count < 1) return 0;
    for (int k = 0; k < count; ++k)
        if (tensors[k].n < 1) return 0;
    return adam_step_workspace(tensors, count);
}

pex_status pex_adam_step(const pex_step_tensor* tensors, int32_t count, pex_adam_variant variant, const pex_adam_params* p,
                         const pex_moment_params* track, float max_norm, double* sum_sq, double* sums, void* workspace, size_t workspace_bytes,
                         pex_stream_t stream)
{
    if (!tensors || !p || !sum_sq || (track && !sums)) return PEX_ERR_NULL;
    if (variant != PEX_ADAM && variant != PEX_MICROADAM && variant != PEX_MICROADAM_VAR && variant != PEX_MICROADAM_MSQ) return PEX_ERR_PHI;
    if (count < 1 || p->step < 1 || p->B < 1 || !(max_norm > 0.f)) return PEX_ERR_SHAPE;
    if ((variant == PEX_MICROADAM_VAR || variant == PEX_MICROADAM_MSQ) && p->B < 2) return PEX_ERR_SHAPE;
    if (track && (track->step < 1 || track->B < 2)) return PEX_ERR_SHAPE;
    for (int k = 0; k < count; ++k) {
        const pex_step_tensor& t = tensors[k];
        if (!t.theta || !t.m || !t.v || !t.S_id || ((variant != PEX_ADAM || track) && !t.S_sq)) return PEX_ERR_NULL;
        if (track && (!t.ema_adam || !t.ema_micro)) return PEX_ERR_NULL;
        if (t.n < 1 || t.n >= ((int64_t)1 << 40)) return PEX_ERR_SHAPE;
        uintptr_t al = (uintptr_t)t.theta | (uintptr_t)t.m | (uintptr_t)t.v | (uintptr_t)t.S_id | (uintptr_t)t.S_sq;
        if (track) al |= (uintptr_t)t.ema_adam | (uintptr_t)t.ema_micro;
        if (al & 15u) return PEX_ERR_ALIGN;
    }
    if (((uintptr_t)sum_sq | (uintptr_t)sums) & 7u) return PEX_ERR_ALIGN;
    if (!workspace || workspace_bytes < adam_step_workspace_least(count)) return PEX_ERR_WORKSPACE;
    if ((uintptr_t)workspace & 15u) return PEX_ERR_ALIGN;
    return launch_adam_step(tensors, count, variant, *p, track, max_norm, sum_sq, sums, workspace, workspace_bytes, (hipStream_t)stream) == hipSuccess
               ? PEX_OK
               : PEX_ERR_HIP;
}

size_t pex_mfma_probe_operand_bytes(void) { return probe_operand_bytes(); }
size_t pex_mfma_probe_sink_floats(int32_t workgroups) { return workgroups < 1 ? 0 : probe_sink_floats(workgroups); }

pex_status pex_mfma_probe(const void* operands, int32_t workgroups, int32_t iters, float* sink, double* flop, pex_stream_t stream)
{
    if (!operands || !sink) return PEX_ERR_NULL;
    if (workgroups < 1 || workgroups > 65536 || iters < 1 || iters > (1 << 24)) return PEX_ERR_SHAPE;
    if (((uintptr_t)operands | (uintptr_t)sink) & 15u) return PEX_ERR_ALIGN;
    if (flop) *flop = probe_flop(workgroups, iters);
    return launch_mfma_probe(operands, workgroups, iters, sink, (hipStream_t)stream) == hipSuccess ? PEX_OK : PEX_ERR_HIP;
}

size_t pex_moment_track_workspace_bytes(int64_t n) { return n < 1 ? 0 : moment_track_workspace(n); }

pex_status pex_moment_track(float* ema_adam, float* ema_micro, const float* S_id, const float* S_sq, int64_t n,
                            const pex_moment_params* p, double* sums, void* workspace, size_t workspace_bytes,
                            pex_stream_t stream)
{
    if (!ema_adam || !ema_micro || !S_id || !S_sq || !p || !sums) return PEX_ERR_NULL;
    if (n < 1 || p->step < 1 || p->B < 2) return PEX_ERR_SHAPE;
    if (((uintptr_t)ema_adam | (uintptr_t)ema_micro | (uintptr_t)S_id | (uintptr_t)S_sq) & 15u) return PEX_ERR_ALIGN;
    if ((uintptr_t)sums & 7u) return PEX_ERR_ALIGN;
    if (!workspace || workspace_bytes < moment_track_workspace(n)) return PEX_ERR_WORKSPACE;
    if ((uintptr_t)workspace & 15u) return PEX_ERR_ALIGN;
    return launch_moment_track(ema_adam, ema_micro, S_id, S_sq, n, *p, sums, (double*)workspace, (hipStream_t)stream) == hipSuccess
               ? PEX_OK
               : PEX_ERR_HIP;
}

pex_status pex_sign_update(float* theta, float* m, const float* S, int64_t n, pex_sign_variant variant, float lr, float beta,
                           float weight_decay, int32_t B, int32_t debias, int64_t step, pex_stream_t stream)
{
    if (!theta || !m || !S) return PEX_ERR_NULL;
    if (variant != PEX_MICROSIGNSGD && variant != PEX_SIGNSGD && variant != PEX_SIGNEMA) return PEX_ERR_PHI;
    if (n < 1 || B < 1 || step < 1) return PEX_ERR_SHAPE;
    if (((uintptr_t)theta | (uintptr_t)m | (uintptr_t)S) & 15u) return PEX_ERR_ALIGN;
    return launch_sign_update(theta, m, S, n, variant, lr, beta, weight_decay, B, debias, step, (hipStream_t)stream) == hipSuccess
               ? PEX_OK
               : PEX_ERR_HIP;
}

pex_status pex_signsgd_update(float* theta, float* m, const float* S_sign, int64_t n, float lr, float beta,
                              float weight_decay, int32_t B, int32_t debias, int64_t step, pex_stream_t stream)
{
    return pex_sign_update(theta, m, S_sign, n, PEX_MICROSIGNSGD, lr, beta, weight_decay, B, debias, step, stream);
}

}  // extern "C"
