// pex_embed.hip -- per-example gradient statistics of an embedding table.
//
// A lookup h[b,t,:] = E[ids[b,t],:] is a dense layer applied to one-hot inputs (Sec. 2.3 with X one-hot), so the
// per-example gradient M_b = onehot(ids_b)^T G_b has, in row v, the sum of the cotangents of the positions of example
// b that hold token v; S = sum_b phi(M_b).  Nothing is contracted: the work is a gather of the rows of G grouped by
// (token, example), so the bound is HBM bandwidth -- G read once, every row of S written once (rows of tokens that do
// not occur are written as zeros), plus the ids.
//
// Everything is deterministic (no floating-point atomics):
//   1. a stable sort of the B*T positions that brings those of a token together; positions enter in the order p = b*T + t, so
//      inside a token's run they stay ordered by example and then by t; ids outside [0, V) (padding) get the key V and are
//      never consumed.  One launch of 256 workgroups that each collect the tokens of one bucket (bucket_sort_kernel); batches and
//      vocabularies too large for that: a least-significant-digit radix sort (8 bits per pass, a counting and a placing
//      launch per pass);
//   2. row_start: where each token's run begins and, at the next index, ends (RowIndex);
//   3. each wave owns 16 consecutive sorted positions and every vocabulary row whose run starts among them: cotangent
//      rows are loaded 16 at a time and added per example, phi is applied whenever the example changes, and the result
//      is added to the row's sums.  Of a row with many positions every wave does the examples that start at its own 16, and the
//      waves' sums are combined in wave order; rows without positions are zero-filled by further workgroups of the same launch.
#include <type_traits>

#include "pex_internal.h"

namespace pex {
namespace {

constexpr int SORT_MAX_BLOCKS = 64;   // workgroups of the sort; a workgroup's tile is a multiple of 1024 keys

template <typename TId>
__device__ __forceinline__ int load_key(const TId* __restrict__ ids, int p, int V)
{
    const int64_t v = (int64_t)ids[p];
    return (v >= 0 && v < (int64_t)V) ? (int)v : V;
}

// Stable least-significant-digit radix sort, 8 bits per pass.  hist[block * 256 + digit] counts the keys of that
// block's tile *of the pass's input* with that digit (the tiles of a later pass hold other keys than those of the
// first, so every pass counts its own input; the counting is in LDS, where many equal keys cost little).
// A tile is a multiple of 1024 keys: 4 rounds of 256 at a time, their loads issued together (8 rounds left half of the 64
// workgroups out at 65536 positions: 4 us more over the four launches).
constexpr int SORT_BATCH = 4;

template <typename TId, bool FIRST>
__global__ __launch_bounds__(256) void sort_hist_kernel(const TId* __restrict__ ids, const int* __restrict__ keys_in, int N, int V,
                                                        int shift, int tile, int* __restrict__ hist)
{
    __shared__ int h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * tile + threadIdx.x;
    for (int r0 = 0; r0 < tile; r0 += 256 * SORT_BATCH) {
        int key[SORT_BATCH];
#pragma unroll
        for (int j = 0; j < SORT_BATCH; ++j) {
            const int64_t p = base + r0 + j * 256;
            key[j] = p < N ? (FIRST ? load_key(ids, (int)p, V) : keys_in[p]) : -1;
        }
#pragma unroll
        for (int j = 0; j < SORT_BATCH; ++j)
            if (key[j] >= 0) atomicAdd(&h[(key[j] >> shift) & 255], 1);
    }
    __syncthreads();
    hist[(int64_t)blockIdx.x * 256 + threadIdx.x] = h[threadIdx.x];
}

// One pass.  A key goes to (keys with a smaller digit) + (keys with the same digit in earlier tiles) + (its rank among
// the keys of its tile with the same digit, in tile order): the first two from the counters (every workgroup adds
// them up for itself: at most 64 tiles), the rank from 8 ballots per key.  FIRST reads the keys from the ids and uses
// the position itself as the value.
template <typename TId, bool FIRST>
__global__ __launch_bounds__(256) void sort_scatter_kernel(const TId* __restrict__ ids, const int* __restrict__ keys_in,
                                                           const int* __restrict__ vals_in, int* __restrict__ keys_out,
                                                           int* __restrict__ vals_out, int N, int V, int shift, int tile, int nblocks,
                                                           const int* __restrict__ hist)
{
    __shared__ int base[256];
    __shared__ int wcnt[4][256];
    __shared__ int wtot[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    {
        int before = 0, total = 0;   // this digit: in earlier tiles, in all tiles
#pragma unroll 8
        for (int b = 0; b < nblocks; ++b) {
            const int c = hist[b * 256 + tid];
            before += b < (int)blockIdx.x ? c : 0;
            total += c;
        }
        int incl = total;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o);
            if (lane >= o) incl += t;
        }
        if (lane == 63) wtot[wave] = incl;
        __syncthreads();
        int smaller = incl - total;   // keys with a smaller digit
        for (int w = 0; w < wave; ++w) smaller += wtot[w];
        base[tid] = smaller + before;
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) wcnt[w][tid] = 0;
    __syncthreads();
    for (int r0 = 0; r0 < tile; r0 += 256 * SORT_BATCH) {
        int keyb[SORT_BATCH], valb[SORT_BATCH];
#pragma unroll
        for (int j = 0; j < SORT_BATCH; ++j) {
            const int64_t idx = (int64_t)blockIdx.x * tile + r0 + j * 256 + tid;
            keyb[j] = -1;
            valb[j] = 0;
            if (idx < N) {
                keyb[j] = FIRST ? load_key(ids, (int)idx, V) : keys_in[idx];
                valb[j] = FIRST ? (int)idx : vals_in[idx];
                if (keyb[j] < 0) keyb[j] = V;   // keys are in [0, V]
            }
        }
#pragma unroll
        for (int j = 0; j < SORT_BATCH; ++j) {
            const bool active = keyb[j] >= 0;
            const int key = keyb[j], val = valb[j];
            const int dg = (key >> shift) & 255;
            // lanes of this wave that are active and hold the same digit
            unsigned long long same = __ballot(active);
#pragma unroll
            for (int bit = 0; bit < 8; ++bit) {
                const bool one = (dg >> bit) & 1;
                const unsigned long long bb = __ballot(one);
                same &= one ? bb : ~bb;
            }
            const int rank = __popcll(same & ((1ull << lane) - 1ull));
            if (active && rank == 0) wcnt[wave][dg] = __popcll(same);
            __syncthreads();
            if (active) {
                int dest = base[dg] + rank;
                for (int w = 0; w < wave; ++w) dest += wcnt[w][dg];
                if (dest >= 0 && dest < N) {   // always true when the counts are those of this very input
                    keys_out[dest] = key;
                    vals_out[dest] = val;
                }
            }
            __syncthreads();
            base[tid] += (wcnt[0][tid] + wcnt[1][tid]) + (wcnt[2][tid] + wcnt[3][tid]);
#pragma unroll
            for (int w = 0; w < 4; ++w) wcnt[w][tid] = 0;
            __syncthreads();
        }
    }
}

// row_start[v] = first index k of the sorted keys with key[k] >= v, for v = 0 .. V (N if there is none).  Position k writes the
// entries between its left neighbour's key and its own, so every entry is written exactly once: short gaps by the position's
// lane, long ones (rare tokens, the end of the vocabulary) by the whole wave.  Called by whole waves, lane l with the
// neighbours prev, cur of a position k (prev >= cur: nothing to write).
__device__ __forceinline__ void fill_row_start(int* __restrict__ row_start, int k, int prev, int cur, int V)
{
    prev = prev < -1 ? -1 : (prev > V ? V : prev);   // keys are in [0, V]; the clamps keep the writes inside the array regardless
    cur = cur > V ? V : cur;
    const int lane = threadIdx.x & 63;
    unsigned long long far = __ballot(cur - prev > 8);
    if (cur - prev <= 8)
        for (int v = prev + 1; v <= cur; ++v) row_start[v] = k;
    while (far) {
        const int l = __builtin_ctzll(far);
        far &= far - 1;
        const int kl = __shfl(k, l), pl = __shfl(prev, l), cl = __shfl(cur, l);
        for (int v = pl + 1 + lane; v <= cl; v += 64) row_start[v] = kl;
    }
}

__global__ __launch_bounds__(256) void row_start_kernel(const int* __restrict__ keys, int N, int V, int* __restrict__ row_start)
{
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool valid = k <= N;
    fill_row_start(row_start, valid ? (int)k : 0, !valid ? 0 : (k == 0 ? -1 : keys[k - 1]), !valid ? 0 : (k == N ? V : keys[k]), V);
}

// Few positions of a vocabulary too large for buckets: the whole radix sort and row_start in one launch of one workgroup, keys
// and positions in LDS.  Same digits, same order: wave i owns a contiguous segment of the positions; counters per (wave, digit) give every key its place.  Bound by the
// latency of its few dozen steps and of writing row_start alone, against the five or seven launches of the kernels above, which take about
// 4.5 us each whatever they do.  Whole calls of 100 / 345 / 630 / 1500 / 2048 positions, by those kernels and by this one, us: V=300000 126 / 70 / 59 /
// 54 / 52, 98 / 56 / 46 / 52 / 54; V=2000000 712 / 289 / 212 / 164 / 150, 556 / 274 / 206 / 184 / 174.
constexpr int SMALL_N = 2048, SMALL_WAVES = 16;

template <typename TId>
__global__ __launch_bounds__(SMALL_WAVES * 64) void sort_small_kernel(const TId* __restrict__ ids, int N, int V, int passes, int* __restrict__ keys_out,
                                                                     int* __restrict__ vals_out, int* __restrict__ row_start)
{
    __shared__ int keys[2][SMALL_N], counts[SMALL_WAVES][256];
    __shared__ uint16_t vals[2][SMALL_N];
    auto key = [&](int buf, int k) -> int& { return keys[buf][k]; };
    auto cnt = [&](int w, int digit) -> int& { return counts[w][digit]; };
    auto val = [&](int buf, int k) -> uint16_t& { return vals[buf][k]; };
    __shared__ int wtot[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int p = tid; p < N; p += SMALL_WAVES * 64) {
        key(0, p) = load_key(ids, p, V);
        val(0, p) = (uint16_t)p;
    }
    const int seg = (N + SMALL_WAVES * 64 - 1) / (SMALL_WAVES * 64) * 64;      // positions per wave, whole batches of 64
    const int lo = wave * seg;
    const int hi = lo + seg < N ? lo + seg : N;
    int cur = 0;
    for (int ps = 0; ps < passes; ++ps) {
        const int shift = 8 * ps;
        for (int t = tid; t < SMALL_WAVES * 256; t += SMALL_WAVES * 64) cnt(t >> 8, t & 255) = 0;
        __syncthreads();
        for (int k = lo + lane; k < hi; k += 64) atomicAdd(&cnt(wave, (key(cur, k) >> shift) & 255), 1);
        __syncthreads();
        // thread t < 256: digit t; its keys start after all smaller digits, wave by wave
        int total = 0, incl = 0;
        if (tid < 256) {
#pragma unroll
            for (int w = 0; w < SMALL_WAVES; ++w) total += cnt(w, tid);
            incl = total;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int t = __shfl_up(incl, o);
                if (lane >= o) incl += t;
            }
            if (lane == 63) wtot[wave] = incl;
        }
        __syncthreads();
        if (tid < 256) {
            int base = incl - total;
            for (int w = 0; w < wave; ++w) base += wtot[w];
#pragma unroll
            for (int w = 0; w < SMALL_WAVES; ++w) {
                const int c = cnt(w, tid);
                cnt(w, tid) = base;
                base += c;
            }
        }
        __syncthreads();
        // batches of 64 in order: rank among the batch's keys of the same digit from 8 ballots, place from the wave's counter,
        // which the first of them moves on
        for (int k0 = lo; k0 < hi; k0 += 64) {
            const bool active = k0 + lane < hi;
            const int kk = active ? key(cur, k0 + lane) : 0;
            const uint16_t vv = active ? val(cur, k0 + lane) : (uint16_t)0;
            const int dg = (kk >> shift) & 255;
            unsigned long long same = __ballot(active);
#pragma unroll
            for (int bit = 0; bit < 8; ++bit) {
                const bool one = (dg >> bit) & 1;
                const unsigned long long bb = __ballot(one);
                same &= one ? bb : ~bb;
            }
            const int rank = __popcll(same & ((1ull << lane) - 1ull));
            const int at = active ? cnt(wave, dg) + rank : 0;
            __builtin_amdgcn_wave_barrier();            // every lane has read its counter (LDS operations of a wave stay in order)
            if (active && rank == 0) cnt(wave, dg) = at + __popcll(same);
            __builtin_amdgcn_wave_barrier();
            if (active && at < N) {
                key(cur ^ 1, at) = kk;
                val(cur ^ 1, at) = vv;
            }
        }
        cur ^= 1;
        __syncthreads();
    }
    for (int k0 = 0; k0 <= N; k0 += SMALL_WAVES * 64) {
        const int k = k0 + tid;
        if (k < N) {
            keys_out[k] = key(cur, k);
            vals_out[k] = val(cur, k);
        }
        const bool valid = k <= N;
        fill_row_start(row_start, valid ? k : 0, !valid ? 0 : (k == 0 ? -1 : key(cur, k - 1)), !valid ? 0 : (k == N ? V : key(cur, k)), V);
    }
}

// The sort by buckets.  Token v belongs to bucket v mod 256 and workgroup b does bucket b alone: it counts the tokens of its
// bucket, places their positions and writes their part of row_start.  Order: by bucket, then by token, then by position --
// consecutive tokens, which are alike in frequency, fall into different buckets.  A wave takes a contiguous part of the positions;
// counters per (wave, token) give every position its place, whatever the frequencies.
//   bucket_sort_kernel<.., false>: one launch.  Every workgroup reads all ids, twice; where its bucket begins it knows from the ids
//     of smaller buckets it meets.  Bound by the instructions of 256 workgroups reading everything: 12 us for 8192 positions, 66
//     for 65536, so it ends at 4096, where two launches take as long.
//   tile_buckets_kernel, bucket_sort_kernel<.., true>: tiles of 1024 positions are first put in bucket order, each by a
//     workgroup of its own; a bucket's workgroup then reads its segment of every tile.  4.8 + 12 us for 65536 positions of Zipf frequencies; 50 where half
//     of them are one token, which one workgroup then places alone.
// (Before: a radix sort with five launches for two 8-bit digits, 30 us.  Whole calls with the rows, identity and square, by that sort and the rows
// kernel of its time / now: B=64 T=1024 V=50257 d=768 115 / 91 us, uniform tokens 93 / 78, half of them one token 175 / 160; B=8 T=512 d=256 59 / 31;
// B=9 T=152 V=2515 d=384 30 / 18; B=128 T=2048 d=256 128 / 84.  A dominant token, which one workgroup places: B=256 T=1024 d=256 with
// 25 / 50 / 90 / 100 % of the positions 215 / 348 / 586 / 864, now 184 / 314 / 542 / 792.)
constexpr int BUCKETS = 256, BUCKET_WAVES = 16, BUCKET_TILE = BUCKET_WAVES * 64, BUCKET_MAX_TILES = 256;
constexpr int BUCKET_MAX_V = BUCKETS * 1024;               // 64 KiB of counters
constexpr int BUCKET_ONE_LAUNCH_N = 4096, BUCKET_MAX_N = BUCKET_MAX_TILES * BUCKET_TILE;

// Where row_start keeps token v: its run is row_start[at(v)] .. row_start[at(v) + 1].  By bucket, or (mask = shift = 0) by token.
struct RowIndex {
    int mask, shift, per_bucket;
    __device__ __forceinline__ int at(int v) const { return (v & mask) * per_bucket + (v >> shift); }
};

// lanes of this wave that are active and hold the same number of `bits` bits
__device__ __forceinline__ unsigned long long same_number(bool active, int x, int bits)
{
    unsigned long long same = __ballot(active);
    for (int b = 0; b < bits; ++b) {
        const bool one = (x >> b) & 1;
        const unsigned long long bb = __ballot(one);
        same &= one ? bb : ~bb;
    }
    return same;
}

// inclusive sum over the lanes of a wave
__device__ __forceinline__ int wave_scan(int x)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(x, o);
        if (lane >= o) x += t;
    }
    return x;
}

// One tile in bucket order, padding left out: keys and positions at the tile's place, off[tile][b] = where bucket b begins in it
template <typename TId>
__global__ __launch_bounds__(BUCKET_TILE) void tile_buckets_kernel(const TId* __restrict__ ids, int N, int V, int* __restrict__ keys_out,
                                                                   int* __restrict__ vals_out, int* __restrict__ off)
{
    __shared__ int counts[BUCKET_WAVES][BUCKETS];
    __shared__ int wtot[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int p = blockIdx.x * BUCKET_TILE + tid;
    for (int t = tid; t < BUCKET_WAVES * BUCKETS; t += BUCKET_TILE) counts[t / BUCKETS][t % BUCKETS] = 0;
    const int key = p < N ? load_key(ids, p, V) : V;
    const bool active = key < V;
    const int b = key & (BUCKETS - 1);
    const unsigned long long same = same_number(active, b, 8);
    const int rank = __popcll(same & ((1ull << lane) - 1ull));
    __syncthreads();
    if (active && rank == 0) counts[wave][b] = __popcll(same);
    __syncthreads();
    int total = 0, incl = 0;
    if (tid < BUCKETS) {
#pragma unroll
        for (int w = 0; w < BUCKET_WAVES; ++w) total += counts[w][tid];
        incl = wave_scan(total);
        if (lane == 63) wtot[wave] = incl;
    }
    __syncthreads();
    if (tid < BUCKETS) {
        int at = incl - total;
        for (int w = 0; w < wave; ++w) at += wtot[w];
        off[blockIdx.x * (BUCKETS + 1) + tid] = at;
        if (tid == BUCKETS - 1) off[blockIdx.x * (BUCKETS + 1) + BUCKETS] = at + total;
#pragma unroll
        for (int w = 0; w < BUCKET_WAVES; ++w) {
            const int c = counts[w][tid];
            counts[w][tid] = at;
            at += c;
        }
    }
    __syncthreads();
    if (active) {
        const int place = blockIdx.x * BUCKET_TILE + counts[wave][b] + rank;
        keys_out[place] = key;
        vals_out[place] = p;
    }
}

// TILED: the segments of tile_buckets_kernel (tiles <= BUCKET_MAX_TILES of them) instead of the ids
template <typename TId, bool TILED>
__global__ __launch_bounds__(BUCKET_TILE) void bucket_sort_kernel(const TId* __restrict__ ids, const int* __restrict__ tile_keys,
                                                                  const int* __restrict__ tile_vals, const int* __restrict__ off, int tiles, int N, int V,
                                                                  int per_bucket, int* __restrict__ keys_out, int* __restrict__ vals_out,
                                                                  int* __restrict__ row_start)
{
    extern __shared__ int counts[];       // [BUCKET_WAVES][per_bucket]
    __shared__ int wsum[2][BUCKET_WAVES];
    __shared__ int seg_at[TILED ? BUCKET_MAX_TILES : 1], seg_src[TILED ? BUCKET_MAX_TILES : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, bucket = blockIdx.x;
    int* mine = counts + wave * per_bucket;
    for (int t = tid; t < BUCKET_WAVES * per_bucket; t += BUCKET_TILE) counts[t] = 0;
    int smaller = 0;      // positions of smaller buckets, this thread's share
    int n = N;            // entries this workgroup reads
    if constexpr (TILED) {
        int len = 0;
        if (tid < tiles) {
            smaller = off[tid * (BUCKETS + 1) + bucket];
            len = off[tid * (BUCKETS + 1) + bucket + 1] - smaller;
            seg_src[tid] = tid * BUCKET_TILE + smaller;
        }
        const int incl = wave_scan(len);
        if (lane == 63) wsum[1][wave] = incl;
        __syncthreads();
        int at = incl - len;
        n = 0;
#pragma unroll
        for (int w = 0; w < BUCKET_MAX_TILES / 64; ++w) {
            if (w < wave) at += wsum[1][w];
            n += wsum[1][w];
        }
        if (tid < tiles) seg_at[tid] = at;
    }
    __syncthreads();
    const int seg = (n + BUCKET_TILE - 1) / BUCKET_TILE * 64;      // entries per wave, whole batches of 64
    const int lo = wave * seg < n ? wave * seg : n, hi = lo + seg < n ? lo + seg : n;
    // entry e: its key and position
    auto entry = [&](int e, int& val) {
        if constexpr (TILED) {
            int t = 0;
            for (int step = BUCKET_MAX_TILES / 2; step > 0; step >>= 1)
                if (t + step < tiles && seg_at[t + step] <= e) t += step;
            const int src = seg_src[t] + (e - seg_at[t]);
            val = tile_vals[src];
            return tile_keys[src];
        } else {
            val = e;
            return load_key(ids, e, V);
        }
    };
    // U batches of 64 from k0 on, their loads in flight together (lanes past the end repeat the last entry)
    auto entries = [&](int k0, auto& key, auto& val) {
        constexpr int U = sizeof(key) / sizeof(int);
        int k[U];
#pragma unroll
        for (int u = 0; u < U; ++u) k[u] = entry(k0 + 64 * u + lane < hi ? k0 + 64 * u + lane : hi - 1, val[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) key[u] = k0 + 64 * u + lane < hi ? k[u] : V;
    };
    auto count = [&](int k0, auto UC) {
        constexpr int U = decltype(UC)::value;
        int key[U], val[U];
        entries(k0, key, val);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int b = key[u] < V ? key[u] & (BUCKETS - 1) : BUCKETS;
            if (!TILED) smaller += b < bucket;
            // (the positions of the first lane's token are one addition: a frequent token's would wait for each other)
            const int first = __builtin_amdgcn_readfirstlane(key[u]);
            const unsigned long long alike = TILED ? __ballot(key[u] == first) : 0;
            if (b == bucket && (!TILED || lane == 0 || key[u] != first)) atomicAdd(&mine[key[u] / BUCKETS], TILED && lane == 0 ? __popcll(alike) : 1);
        }
    };
    constexpr std::integral_constant<int, 8> U8{};
    constexpr std::integral_constant<int, 1> U1{};
    int at0 = lo;
    for (; at0 + 64 * 7 < hi; at0 += 64 * 8) count(at0, U8);
    for (; at0 < hi; at0 += 64) count(at0, U1);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) smaller += __shfl_xor(smaller, o);
    if (lane == 0) wsum[0][wave] = smaller;
    __syncthreads();
    // thread t: the bucket's token t; its run begins after all smaller ones, wave by wave
    int total = 0;
    if (tid < per_bucket)
#pragma unroll
        for (int w = 0; w < BUCKET_WAVES; ++w) total += counts[w * per_bucket + tid];
    const int incl = wave_scan(total);
    if (lane == 63) wsum[1][wave] = incl;
    __syncthreads();
    int at = incl - total, end = 0;
#pragma unroll
    for (int w = 0; w < BUCKET_WAVES; ++w) {
        at += wsum[0][w] + (w < wave ? wsum[1][w] : 0);
        end += wsum[0][w] + wsum[1][w];
    }
    if (tid < per_bucket) {
        row_start[bucket * per_bucket + tid] = at;
#pragma unroll
        for (int w = 0; w < BUCKET_WAVES; ++w) {
            const int c = counts[w * per_bucket + tid];
            counts[w * per_bucket + tid] = at;
            at += c;
        }
    }
    if (bucket == BUCKETS - 1) {          // the last run's end, and the positions of padding
        if (tid == 0) row_start[BUCKETS * per_bucket] = end;
        for (int k = end + tid; k < N; k += BUCKET_TILE) {
            keys_out[k] = V;
            vals_out[k] = 0;
        }
    }
    __syncthreads();
    int bits = 0;
    while ((per_bucket - 1) >> bits) ++bits;
    auto place_batches = [&](int k0, auto UC) {
        constexpr int U = decltype(UC)::value;
        int key[U], val[U];
        entries(k0, key, val);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool match = key[u] < V && (key[u] & (BUCKETS - 1)) == bucket;
            unsigned long long todo = __ballot(match), same = 0;
            if (todo == 0) continue;
            // batches of 64 in order: rank among the batch's positions of the same token, place from the wave's counter, which the
            // first of them moves on.  Up to four tokens (a frequent one among others) one by one, more by their bits.
            const int token = match ? key[u] / BUCKETS : 0;
            for (int i = 0; i < 4 && todo; ++i) {
                const unsigned long long m = __ballot(match && key[u] == __builtin_amdgcn_readlane(key[u], __builtin_ctzll(todo)));
                if ((m >> lane) & 1) same = m;
                todo &= ~m;
            }
            if (todo) same = same_number(match, token, bits);
            const int rank = __popcll(same & ((1ull << lane) - 1ull));
            const int place = match ? mine[token] + rank : 0;
            __builtin_amdgcn_wave_barrier();            // every lane has read its counter (LDS operations of a wave stay in order)
            if (match && rank == 0) mine[token] = place + __popcll(same);
            __builtin_amdgcn_wave_barrier();
            if (match && place < N) {
                keys_out[place] = key[u];
                vals_out[place] = val[u];
            }
        }
    };
    at0 = lo;
    for (; at0 + 64 * 7 < hi; at0 += 64 * 8) place_batches(at0, U8);
    for (; at0 < hi; at0 += 64) place_batches(at0, U1);
}

// What a lane loads from a cotangent row: four columns (fp32 16 bytes, bf16 8 bytes), kept as loaded until they are added:
// widening bf16 early would double the registers a lane holds in flight.  Four columns per lane make the fp32 stores of a
// wave dense (16 bytes per lane, 1 KiB per instruction); eight bf16 columns per lane would leave every store instruction
// writing half of each 32 bytes.
// ALIGN = the largest of 4, 2, 1 that divides the row length, 0 for rows shorter than four columns.  Rows of any length from
// four on are whole chunks: the last lane takes the row's last four columns, whoever else has some of them (the same sums in
// the same order).  A chunk is one load whatever its address.  (Element by element, one column per lane, before: V=50257, d=767,
// B=64 T=1024 288 us, 161 with two aligned loads; V=40529, d=206, B=6 T=105 108 us, 43 together with the sort of one launch.)
constexpr int CH = 4;

template <typename TIn, int ALIGN>
struct Chunk {
    typedef __attribute__((ext_vector_type(4))) unsigned int u4;
    typedef __attribute__((ext_vector_type(2))) unsigned int u2;
    typedef u4 __attribute__((aligned(4))) u4_u;
    typedef u2 __attribute__((aligned(2))) u2_u;
    static constexpr bool BF16 = sizeof(TIn) == 2;
    static constexpr int WORDS = !BF16 || ALIGN == 0 ? 4 : 2;
    typedef typename std::conditional<WORDS == 4, u4, u2>::type Raw;
    // columns col .. col+3 of `row` (of length d)
    static __device__ __forceinline__ Raw load(const TIn* row, int64_t col, int64_t d)
    {
        const TIn* p = row + col;
        if constexpr (ALIGN == 0) {          // fewer than four columns: the last one stands in for those beyond
            Raw z;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const TIn x = p[e < (int)d ? e : (int)d - 1];
                z[e] = __builtin_bit_cast(typename std::conditional<BF16, unsigned short, unsigned int>::type, x);
            }
            return z;
        } else if constexpr (!BF16) return *(const u4_u*)p;
        else if constexpr (ALIGN == 4) return *(const u2*)p;
        else return *(const u2_u*)p;
    }
    static __device__ __forceinline__ void add_to(float (&acc)[CH], const Raw& raw)
    {
        if constexpr (WORDS == 4) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += __uint_as_float(BF16 ? raw[e] << 16 : raw[e]);
        } else {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                acc[2 * e] += __uint_as_float(raw[e] << 16);
                acc[2 * e + 1] += __uint_as_float(raw[e] & 0xffff0000u);
            }
        }
    }
};

// Four columns, in rows shorter than that d of them.  OUTPUT: rows of S, which nothing reads soon: past the caches (two
// statistics of a GPT-2 vocabulary are 309 MB; 141 -> 130 us)
template <int ALIGN, bool OUTPUT = true>
__device__ __forceinline__ void store_chunk(float* p, const float (&v)[CH], int64_t d)
{
    typedef __attribute__((ext_vector_type(4))) float f4;
    typedef f4 __attribute__((aligned(4))) f4_u;
    const f4 q = {v[0], v[1], v[2], v[3]};
    if constexpr (ALIGN == 0) {
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (e < (int)d) p[e] = v[e];
    } else if constexpr (OUTPUT) __builtin_nontemporal_store(q, (f4_u*)p);
    else *(f4_u*)p = q;
}

// first column of the chunk at `col` (a multiple of four): the row's last chunk ends with the row
template <int ALIGN>
__device__ __forceinline__ int64_t chunk_start(int64_t col, int64_t d)
{
    return ALIGN != 0 && ALIGN != 4 && col + CH > d ? d - CH : col;
}

// waves of a workgroup: two of 12 or three of 8 share a compute unit where 16 left the first half of a frequent token's run waiting
// for the second (141 -> 135 us; 4 waves 6 us slower than 8); a slice of partial sums is EMB_WAVES * EMB_U positions, so fewer
// waves cost workspace
constexpr int EMB_WAVES = 12;
constexpr int EMB_ZROWS = 8;     // vocabulary rows a zero-fill wave looks at
constexpr int EMB_U = 16;        // sorted positions a wave owns = cotangent rows a lane keeps in flight
// A vocabulary row with at most so many positions is done by the wave it starts at; of a longer one each wave does its own examples.  Few
// workgroups wait for the longest chain of such rows, sixteen at a time, of a wave: EMB_U (no less: two long runs must not start at one wave's
// positions).  A full chip does not, nor does one with a workgroup a unit that mostly writes a large table, and every row done together costs a
// pass through LDS: 64, whose positions a lane each reads ahead.  The time of whole calls with 64 over that with 16, 125 drawn ones of 129 to 912
// workgroups, in the mean: at most 256 workgroups 1.08 up to 2^24 entries of the table, 1.00 (1.00 to 1.02) beyond; 257 to 512 1.05 up to 2^23, 1.00
// (0.97 to 1.05) up to 2^24 and 0.99 (0.98 to 1.00) beyond; more 1.02 up to 2^23, which this leaves, and 0.99 (0.97 to 1.02) beyond.  B=64 T=1000
// V=2000 d=200 (334 workgroups) 37.9 and 34.3 us, B=40 T=600 V=9000 d=512 (250) 30.7 and 28.3; B=64 T=700 V=40000 d=768 (702) 71.7 and 72.1.
inline int embed_alone(int64_t workgroups, int64_t entries) { return workgroups > 2 * 256 || (workgroups > 256 && entries > ((int64_t)1 << 24)) ? 64 : EMB_U; }

struct RowSums {
    float id[CH], sq[CH], sg[CH];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int e = 0; e < CH; ++e) id[e] = sq[e] = sg[e] = 0.f;
    }
};

// Accumulates the cotangent rows of one vocabulary row, example by example: acc holds the running sum of the current
// example, phi(acc) goes to the row's sums when the example changes.
template <typename TIn, int ALIGN, int WANT>
struct RowAccumulator {
    RowSums sums;
    float acc[CH];
    int example;     // whose sum acc holds, -1: none
    __device__ __forceinline__ void start()
    {
        sums.clear();
#pragma unroll
        for (int e = 0; e < CH; ++e) acc[e] = 0.f;
        example = -1;
    }
    __device__ __forceinline__ void fold()
    {
#pragma unroll
        for (int e = 0; e < CH; ++e) {
            if (WANT & 1) sums.id[e] += acc[e];
            if (WANT & 2) sums.sq[e] = fmaf(acc[e], acc[e], sums.sq[e]);
            if (WANT & 4) sums.sg[e] += (float)((acc[e] > 0.f) - (acc[e] < 0.f));
            acc[e] = 0.f;
        }
    }
    // `of` is uniform over the wave
    __device__ __forceinline__ void add(int of, const typename Chunk<TIn, ALIGN>::Raw& raw)
    {
        if (of != example) finish();
        example = of;
        Chunk<TIn, ALIGN>::add_to(acc, raw);
    }
    __device__ __forceinline__ void finish()
    {
        if (example >= 0) fold();
        example = -1;
    }
};

// WANT: bit 0 identity, bit 1 square, bit 2 sign.
// grid = chunk workgroups of every block of 64 * CH columns, then the zero-fill workgroups: the chunks are the long poles, the
// zero fill runs under their tail (with the column blocks one after the other, each with its own tail, 149 against 141 us).
//   chunk workgroup: wave i owns the sorted positions [c0, c0 + EMB_U) and with them every vocabulary row whose run
//     starts there, and, of a run longer than `alone`, the examples that start there (each may continue past c0 + EMB_U).  It
//     loads EMB_U cotangent rows at a time whatever rows and examples they belong to, then adds them in order; sums of long runs
//     go to LDS, where the wave a run starts at combines them after the one barrier.
//     Small calls are bound by one wave's instructions: its lookups take 1.3 us, its own sixteen rows 3.6 (at most 6), sixteen more of the
//     run it is in 2 to 3 (measured inside the kernel).  All long runs of a workgroup are done side by side, the positions behind a
//     wave's own are read ahead with the first load, nothing searches for the bounds of examples, one copy of the code adds a row.
//   zero-fill workgroup: wave i looks at EMB_ZROWS vocabulary rows and writes zeros to those without positions.
template <typename TIn, int ALIGN, int WANT>
__global__ __launch_bounds__(EMB_WAVES * 64) void embed_rows_kernel(const TIn* __restrict__ G, const int* __restrict__ row_start,
                                                                    const int* __restrict__ keys, const int* __restrict__ pos,
                                                                    int N, int V, int T, int64_t d, RowIndex index, int alone, int chunk_groups,
                                                                    int colblocks, float* __restrict__ partial, float* __restrict__ S_id,
                                                                    float* __restrict__ S_sq, float* __restrict__ S_sg)
{
    typedef Chunk<TIn, ALIGN> Ck;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool zero_fill = (int)blockIdx.x >= chunk_groups * colblocks;
    const int group = zero_fill ? (int)blockIdx.x - chunk_groups * colblocks : (int)blockIdx.x / colblocks;
    const int64_t col0 = ((int64_t)(blockIdx.x % colblocks) * 64 + lane) * CH;
    const bool col_ok = col0 < d;
    const int64_t col = chunk_start<ALIGN>(col0, d);
    auto store_row = [&](int v, const RowSums& sums) {
        if (!col_ok) return;
        const int64_t o = (int64_t)v * d + col;
        if (WANT & 1) store_chunk<ALIGN>(S_id + o, sums.id, d);
        if (WANT & 2) store_chunk<ALIGN>(S_sq + o, sums.sq, d);
        if (WANT & 4) store_chunk<ALIGN>(S_sg + o, sums.sg, d);
    };

    if (zero_fill) {
        // whole rows, all column blocks by the same wave: an empty row is one contiguous run of d floats, and empty
        // rows are often neighbours
        const int v = (group * EMB_WAVES + wave) * EMB_ZROWS + lane;
        const int r = v < V ? index.at(v) : 0;
        const bool empty = lane < EMB_ZROWS && v < V && row_start[r] == row_start[r + 1];
        unsigned long long todo = __ballot(empty);
        RowSums zeros;
        zeros.clear();
        while (todo) {
            const int l = __builtin_ctzll(todo);
            todo &= todo - 1;
            const int64_t o = (int64_t)(v - lane + l) * d;
            for (int64_t c0 = (int64_t)lane * CH; c0 < d; c0 += 64 * CH) {
                const int64_t c = chunk_start<ALIGN>(c0, d);
                if (WANT & 1) store_chunk<ALIGN>(S_id + o + c, zeros.id, d);
                if (WANT & 2) store_chunk<ALIGN>(S_sq + o + c, zeros.sq, d);
                if (WANT & 4) store_chunk<ALIGN>(S_sg + o + c, zeros.sg, d);
            }
        }
        return;
    }

    constexpr int NSTAT = (WANT & 1) + (WANT >> 1 & 1) + (WANT >> 2 & 1);
    typedef __attribute__((ext_vector_type(4))) float f4;
    // sums of the long runs at wave i's positions: slot 0 of the one that goes on from before them, slot 1 of the one that starts there
    __shared__ f4 comb[EMB_WAVES][2][NSTAT][64];
    const int64_t c0l = ((int64_t)group * EMB_WAVES + wave) * EMB_U;
    const int c0 = c0l < N ? (int)c0l : N;
    const int c1 = c0 + EMB_U < N ? c0 + EMB_U : N;

    // Lane u < EMB_U looks up position c0 + u: its token and the extent of the token's run; the 64 positions behind are read ahead, a
    // lane each.  Loaded are: positions of runs that start here, and of a long run that goes on from before the examples that start here.
    const int k = c0 + lane;
    const bool valid = lane < EMB_U && k < N;
    int key = V, p = -1, rs = 0, re = 0;
    if (valid) { key = keys[k]; p = pos[k]; }
    const int before = c0 > 0 ? pos[c0 - 1] : -1;
    int behind = c1 + lane < N ? pos[c1 + lane] : -1;
    key = key < 0 ? V : (key > V ? V : key);
    if (valid && key < V) { const int r = index.at(key); rs = row_start[r]; re = row_start[r + 1]; }
    re = re > N ? N : re;
    const bool is_long = re - rs > alone;
    const int of = p / T;
    const bool mine = rs >= c0 || (is_long && (before < 0 || of > before / T));
    const int p_ld = (valid && key < V && mine && p >= 0 && p < N) ? p : -1;
    const unsigned long long starts = __ballot(valid && key < V && is_long && rs == k);         // at most one among EMB_U positions
    const int row_before = __builtin_amdgcn_readfirstlane(valid && key < V && is_long && rs < c0 ? key : -1);
    const int from_before = __builtin_amdgcn_readfirstlane(rs), to_before = __builtin_amdgcn_readfirstlane(re);
    const int start_lane = starts ? (int)__builtin_ctzll(starts) : 0;
    const int row_starting = starts ? __builtin_amdgcn_readlane(key, start_lane) : -1, to_starting = __builtin_amdgcn_readlane(re, start_lane);

    RowAccumulator<TIn, ALIGN, WANT> ra;
    ra.start();
    int cur_v = -1;      // the row being accumulated
    auto keep = [&](int slot) {
        int n = 0;
        if (WANT & 1) comb[wave][slot][n++][lane] = f4{ra.sums.id[0], ra.sums.id[1], ra.sums.id[2], ra.sums.id[3]};
        if (WANT & 2) comb[wave][slot][n++][lane] = f4{ra.sums.sq[0], ra.sums.sq[1], ra.sums.sq[2], ra.sums.sq[3]};
        if (WANT & 4) comb[wave][slot][n++][lane] = f4{ra.sums.sg[0], ra.sums.sg[1], ra.sums.sg[2], ra.sums.sg[3]};
    };
    auto close = [&]() {
        if (cur_v < 0) return;
        ra.finish();
        if (cur_v == row_before) keep(0);
        else if (cur_v == row_starting) keep(1);
        else store_row(cur_v, ra.sums);
        ra.sums.clear();
    };
    if (row_before >= 0) keep(0);      // zeros, where no example of it starts here
    // EMB_U cotangent rows, loaded at once whatever rows and examples they belong to, then added one after the other by one copy of the
    // code, whose index into the registers is uniform over the wave: of 16 copies, each with the ends of examples and rows, a wave runs
    // through cold code once (own sixteen rows of the slowest wave 6 us instead of 9; B=17 T=38 V=3662 d=192 16.0 -> 15.0 us).
    constexpr int WORDS = Ck::WORDS, PER = 32 / WORDS, PARTS = EMB_U / PER;
    typedef __attribute__((ext_vector_type(32))) unsigned int u32;
    u32 data[PARTS];
    const int64_t col_ld = col_ok ? col : 0;
    auto load_rows = [&](int p_of_lane, int first) {       // rows of the positions that lanes first .. first + EMB_U - 1 hold (negative: none, row 0)
#pragma unroll
        for (int u = 0; u < EMB_U; ++u) {
            const int q = __builtin_amdgcn_readlane(p_of_lane, first + u);
            if (q < 0) continue;
            const typename Ck::Raw raw = Ck::load(G + (int64_t)q * d, col_ld, d);
#pragma unroll
            for (int e = 0; e < WORDS; ++e) data[u / PER][u % PER * WORDS + e] = raw[e];
        }
    };
    auto row = [&](const u32& part, int which) {
        typename Ck::Raw raw;
#pragma unroll
        for (int e = 0; e < WORDS; ++e) raw[e] = part[which * WORDS + e];
        return raw;
    };
    load_rows(p_ld, 0);
#pragma unroll
    for (int part = 0; part < PARTS; ++part)
#pragma unroll 1
        for (int i = 0; i < PER; ++i) {
            const int q = __builtin_amdgcn_readlane(p_ld, part * PER + i), v = __builtin_amdgcn_readlane(key, part * PER + i);
            if (q < 0) continue;
            if (v != cur_v) {
                close();
                cur_v = v;
            }
            ra.add(__builtin_amdgcn_readlane(of, part * PER + i), row(data[part], i));
        }
    // what is left of the last position's run: all of it, or of a long one the rest of the example
    if (__builtin_amdgcn_readlane(p_ld, EMB_U - 1) >= 0) {
        const int run_end = __builtin_amdgcn_readlane(re, EMB_U - 1), last_of = __builtin_amdgcn_readlane(of, EMB_U - 1);
        const bool whole = __builtin_amdgcn_readlane((int)is_long, EMB_U - 1) == 0;
        for (int k0 = c1;; k0 += 64) {
            const int behind_of = behind / T;
            const unsigned long long rest = ~__ballot(k0 + lane < run_end && (whole || behind_of == last_of));
            const int n = rest ? (int)__builtin_ctzll(rest) : 64;
            for (int u0 = 0; u0 < n; u0 += EMB_U) {
                load_rows(lane < n ? behind : -1, u0);
#pragma unroll
                for (int u = 0; u < EMB_U; ++u)      // (one row's, short: 16 copies)
                    if (u0 + u < n)
                        ra.add(__builtin_amdgcn_readlane(behind_of, u0 + u), row(data[u / PER], u % PER));
            }
            if (n < 64) break;
            behind = k0 + 64 + lane < N ? pos[k0 + 64 + lane] : -1;
        }
    }
    close();
    __syncthreads();

    // A long run's sums of the waves it covers, in wave order, by the wave it starts at (by the first one if it goes on from before the
    // workgroup's positions [sc0, sc1)).  A run that lies inside these is finished here; of any other the sums go to `partial`
    // (slot 0: goes on from before, slot 1: starts here and goes on) for embed_combine_kernel.
    const int64_t sc0 = (int64_t)group * (EMB_WAVES * EMB_U);
    const int64_t sc1 = sc0 + EMB_WAVES * EMB_U < N ? sc0 + EMB_WAVES * EMB_U : N;
    auto combine = [&](int v, int slot, bool goes_on_from, int end) {
        if (!col_ok) return;
        f4 sum[NSTAT];
#pragma unroll
        for (int n = 0; n < NSTAT; ++n) sum[n] = comb[wave][slot][n][lane];
        for (int w = wave + 1; w < EMB_WAVES && sc0 + w * EMB_U < end; ++w)
#pragma unroll
            for (int n = 0; n < NSTAT; ++n) sum[n] += comb[w][0][n][lane];
        const bool inside = !goes_on_from && end <= sc1;
        int n = 0;
#pragma unroll
        for (int stat = 0; stat < 3; ++stat) {
            if (!(WANT & (1 << stat))) continue;
            const float x[CH] = {sum[n][0], sum[n][1], sum[n][2], sum[n][3]};
            ++n;
            if (inside) store_chunk<ALIGN>((stat == 0 ? S_id : stat == 1 ? S_sq : S_sg) + (int64_t)v * d + col, x, d);
            else store_chunk<ALIGN, false>(partial + (((int64_t)group * 2 + (goes_on_from ? 0 : 1)) * 3 + stat) * d + col, x, d);
        }
    };
    if (wave == 0 && row_before >= 0 && from_before < sc0) combine(row_before, 0, true, to_before);
    if (row_starting >= 0) combine(row_starting, 1, false, to_starting);
}

// Finishes the long runs that span several workgroups of embed_rows_kernel: the workgroup-sized slice s in which such a
// run starts adds up the partial sums of the slices the run covers, in slice order, and stores the row.
// grid = (slices, column blocks), one wave each.
template <int ALIGN, int WANT>
__global__ __launch_bounds__(64) void embed_combine_kernel(const int* __restrict__ row_start, const int* __restrict__ keys, int N, int V,
                                                           int64_t d, RowIndex index, int alone, const float* __restrict__ partial,
                                                           float* __restrict__ S_id, float* __restrict__ S_sq, float* __restrict__ S_sg)
{
    constexpr int SLICE = EMB_WAVES * EMB_U;
    const int64_t sc0 = (int64_t)blockIdx.x * SLICE, sc1 = sc0 + SLICE;
    if (sc1 >= N) return;   // nothing goes on past the last slice
    const int key = keys[sc1 - 1];
    if (key < 0 || key >= V) return;
    const int rs = row_start[index.at(key)], re = row_start[index.at(key) + 1];
    if (!(rs >= sc0 && re > sc1 && re <= N && re - rs > alone)) return;
    const int64_t col0 = ((int64_t)blockIdx.y * 64 + threadIdx.x) * CH;
    if (col0 >= d) return;
    const int64_t col = chunk_start<ALIGN>(col0, d);
    // (eight slices' partial sums are loaded together: a run of many slices -- a token that fills half of a batch of 65536 crosses
    // 170 -- is a chain of additions, not of loads: 57 -> 13 us there)
    float sum[3][CH];
    auto take = [&](int64_t slice, int slot, auto UC, bool first) {      // this and the following slices
        constexpr int U = decltype(UC)::value;
        float v[U][3][CH];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float* pr = partial + (((slice + u) * 2 + slot) * 3) * d + col;
#pragma unroll
            for (int o = 0; o < 3; ++o)
                if (WANT & (1 << o))
#pragma unroll
                    for (int e = 0; e < CH; ++e) v[u][o][e] = ALIGN != 0 || e < (int)d ? pr[o * d + e] : 0.f;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int o = 0; o < 3; ++o)
                if (WANT & (1 << o))
#pragma unroll
                    for (int e = 0; e < CH; ++e) sum[o][e] = first ? v[u][o][e] : sum[o][e] + v[u][o][e];
    };
    constexpr std::integral_constant<int, 1> U1{};
    constexpr std::integral_constant<int, 8> U8{};
    take(blockIdx.x, 1, U1, true);
    const int64_t end = (re + SLICE - 1) / SLICE;      // past the slice the run ends in
    int64_t sl = (int64_t)blockIdx.x + 1;
    for (; sl + 8 <= end; sl += 8) take(sl, 0, U8, false);
    for (; sl < end; ++sl) take(sl, 0, U1, false);
    const int64_t o = (int64_t)key * d + col;
    if (WANT & 1) store_chunk<ALIGN>(S_id + o, sum[0], d);
    if (WANT & 2) store_chunk<ALIGN>(S_sq + o, sum[1], d);
    if (WANT & 4) store_chunk<ALIGN>(S_sg + o, sum[2], d);
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Where the workspace keeps what (byte offsets).  The partial sums come last: two of three statistics per slice of EMB_WAVES * EMB_U
// positions, for runs that cross slices.
struct EmbedLayout {
    int passes, tile, nblocks;
    size_t hist, keys_a, vals_a, keys_b, vals_b, row_start, partial, total;
};

// by_bucket: `hist` holds the offsets of tile_buckets_kernel; up to BUCKET_ONE_LAUNCH_N positions need no more than the radix sort does
// (256 * ceil(V / 256) + 1 entries of row_start are at most 1020 bytes more than its V + 2, its counters and buffers 1536)
EmbedLayout embed_layout(int64_t N, int64_t V, int64_t d, bool by_bucket)
{
    EmbedLayout L;
    int bits = 0;
    while (((int64_t)1 << bits) <= V) ++bits;   // the largest key is V
    L.passes = (bits + 7) / 8;
    if (L.passes < 1) L.passes = 1;
    int64_t tile = (N + SORT_MAX_BLOCKS - 1) / SORT_MAX_BLOCKS;
    tile = (tile + 1023) / 1024 * 1024;
    L.tile = (int)tile;
    L.nblocks = (int)((N + tile - 1) / tile);
    const bool one_launch = by_bucket && N <= BUCKET_ONE_LAUNCH_N;
    const size_t list = align256((size_t)N * sizeof(int)), tiles = (size_t)(N + BUCKET_TILE - 1) / BUCKET_TILE;
    size_t o = 0;
    L.hist = o; o += one_launch ? 0 : by_bucket ? align256(tiles * (BUCKETS + 1) * sizeof(int)) : align256((size_t)256 * L.nblocks * sizeof(int));
    L.keys_a = o; o += list;
    L.vals_a = o; o += list;
    L.keys_b = o; o += one_launch ? 0 : list;
    L.vals_b = o; o += one_launch ? 0 : list;
    L.row_start = o; o += align256((by_bucket ? (size_t)BUCKETS * (size_t)((V + BUCKETS - 1) / BUCKETS) + 1 : (size_t)(V + 2)) * sizeof(int));
    const int64_t slices = (N + EMB_WAVES * EMB_U - 1) / (EMB_WAVES * EMB_U);
    L.partial = o; o += align256((size_t)slices * 2 * 3 * d * sizeof(float));
    L.total = o;
    return L;
}

// By buckets: one launch while 256 readers of the ids cost less than a second one, two while a tile has a lane
inline bool sorts_by_bucket(int64_t N, int64_t V) { return N <= BUCKET_MAX_N && V <= BUCKET_MAX_V; }

template <typename TId>
hipError_t sort_positions(const TId* ids, int N, int V, bool by_bucket, const EmbedLayout& L, char* ws, const int** keys, const int** vals,
                          RowIndex* index, hipStream_t stream)
{
    int* hist = (int*)(ws + L.hist);
    int* ka = (int*)(ws + L.keys_a);
    int* va = (int*)(ws + L.vals_a);
    int* kb = (int*)(ws + L.keys_b);
    int* vb = (int*)(ws + L.vals_b);
    int* row_start = (int*)(ws + L.row_start);
    if (by_bucket) {
        const int per_bucket = (V + BUCKETS - 1) / BUCKETS, tiles = (N + BUCKET_TILE - 1) / BUCKET_TILE;
        const size_t lds = (size_t)BUCKET_WAVES * per_bucket * sizeof(int);
        *index = RowIndex{BUCKETS - 1, 8, per_bucket};
        *keys = ka;
        *vals = va;
        if (N <= BUCKET_ONE_LAUNCH_N) {
            bucket_sort_kernel<TId, false><<<dim3(BUCKETS), dim3(BUCKET_TILE), lds, stream>>>(ids, nullptr, nullptr, nullptr, 0, N, V, per_bucket, ka, va, row_start);
        } else {
            tile_buckets_kernel<TId><<<dim3(tiles), dim3(BUCKET_TILE), 0, stream>>>(ids, N, V, kb, vb, hist);
            bucket_sort_kernel<TId, true><<<dim3(BUCKETS), dim3(BUCKET_TILE), lds, stream>>>(ids, kb, vb, hist, tiles, N, V, per_bucket, ka, va, row_start);
        }
        return hipGetLastError();
    }
    *index = RowIndex{0, 0, 0};
    if (N <= SMALL_N) {
        sort_small_kernel<TId><<<dim3(1), dim3(SMALL_WAVES * 64), 0, stream>>>(ids, N, V, L.passes, ka, va, row_start);
        *keys = ka;
        *vals = va;
        return hipGetLastError();
    }
    const dim3 grid(L.nblocks), block(256);
    const int* kin = nullptr;
    const int* vin = nullptr;
    int* kout = ka;
    int* vout = va;
    for (int ps = 0; ps < L.passes; ++ps) {
        if (ps == 0) {
            sort_hist_kernel<TId, true><<<grid, block, 0, stream>>>(ids, nullptr, N, V, 0, L.tile, hist);
            sort_scatter_kernel<TId, true><<<grid, block, 0, stream>>>(ids, nullptr, nullptr, kout, vout, N, V, 0, L.tile, L.nblocks, hist);
        } else {
            sort_hist_kernel<TId, false><<<grid, block, 0, stream>>>(ids, kin, N, V, 8 * ps, L.tile, hist);
            sort_scatter_kernel<TId, false><<<grid, block, 0, stream>>>(ids, kin, vin, kout, vout, N, V, 8 * ps, L.tile, L.nblocks, hist);
        }
        kin = kout; vin = vout;
        kout = (kout == ka) ? kb : ka;
        vout = (vout == va) ? vb : va;
    }
    *keys = kin;
    *vals = vin;
    row_start_kernel<<<dim3((unsigned)(((int64_t)N + 1 + 255) / 256)), dim3(256), 0, stream>>>(kin, N, V, row_start);
    return hipGetLastError();
}

template <typename TIn, int ALIGN, int WANT>
hipError_t launch_rows(const TIn* G, const int* row_start, const int* keys, const int* pos, int N, int V, int T, int64_t d,
                       RowIndex index, float* partial, float* S_id, float* S_sq, float* S_sg, hipStream_t stream)
{
    const int64_t per_group = (int64_t)EMB_WAVES * EMB_U;
    const int chunk_groups = (int)((N + per_group - 1) / per_group);
    const int zero_groups = (int)(((int64_t)V + EMB_WAVES * EMB_ZROWS - 1) / (EMB_WAVES * EMB_ZROWS));
    const unsigned colblocks = (unsigned)((d + 64 * CH - 1) / (64 * CH));
    const int alone = embed_alone((int64_t)chunk_groups * colblocks, (int64_t)V * d);
    embed_rows_kernel<TIn, ALIGN, WANT><<<dim3((unsigned)chunk_groups * colblocks + (unsigned)zero_groups), dim3(EMB_WAVES * 64), 0, stream>>>(
        G, row_start, keys, pos, N, V, T, d, index, alone, chunk_groups, (int)colblocks, partial, S_id, S_sq, S_sg);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || chunk_groups == 1) return e;       // no run leaves a single slice
    embed_combine_kernel<ALIGN, WANT><<<dim3((unsigned)chunk_groups, colblocks), dim3(64), 0, stream>>>(row_start, keys, N, V, d, index, alone, partial,
                                                                                                   S_id, S_sq, S_sg);
    return hipGetLastError();
}

template <typename TIn, int ALIGN>
hipError_t launch_rows_want(uint32_t want, const TIn* G, const int* rs, const int* keys, const int* pos, int N, int V, int T, int64_t d, RowIndex ix, float* pr, float* a,
                            float* q, float* g, hipStream_t st)
{
    switch (want) {
    case 1: return launch_rows<TIn, ALIGN, 1>(G, rs, keys, pos, N, V, T, d, ix, pr, a, q, g, st);
    case 2: return launch_rows<TIn, ALIGN, 2>(G, rs, keys, pos, N, V, T, d, ix, pr, a, q, g, st);
    case 3: return launch_rows<TIn, ALIGN, 3>(G, rs, keys, pos, N, V, T, d, ix, pr, a, q, g, st);
    case 4: return launch_rows<TIn, ALIGN, 4>(G, rs, keys, pos, N, V, T, d, ix, pr, a, q, g, st);
    case 5: return launch_rows<TIn, ALIGN, 5>(G, rs, keys, pos, N, V, T, d, ix, pr, a, q, g, st);
    case 6: return launch_rows<TIn, ALIGN, 6>(G, rs, keys, pos, N, V, T, d, ix, pr, a, q, g, st);
    default: return launch_rows<TIn, ALIGN, 7>(G, rs, keys, pos, N, V, T, d, ix, pr, a, q, g, st);
    }
}

}  // namespace

// (what a call needs: the radix sort's, with which a smaller workspace than the query's makes do)
size_t embed_workspace_least(int64_t B, int64_t T, int64_t V, int64_t d) { return embed_layout(B * T, V, d, false).total; }

size_t embed_workspace(int64_t B, int64_t T, int64_t V, int64_t d)
{
    const size_t least = embed_workspace_least(B, T, V, d);
    const size_t by_bucket = sorts_by_bucket(B * T, V) ? embed_layout(B * T, V, d, true).total : 0;
    return by_bucket > least ? by_bucket : least;
}

hipError_t launch_embed_stat(const void* ids, int ids_bytes, const void* G, int64_t B, int64_t T, int64_t V, int64_t d,
                             pex_dtype dt, uint32_t want, float* S_id, float* S_sq, float* S_sign, void* workspace, size_t workspace_bytes,
                             hipStream_t stream)
{
    const int N = (int)(B * T);
    bool by_bucket = sorts_by_bucket(N, V);
    EmbedLayout L = embed_layout(N, V, d, by_bucket);
    if (by_bucket && workspace_bytes < L.total) L = embed_layout(N, V, d, by_bucket = false);
    char* ws = (char*)workspace;
    const int* keys = nullptr;
    const int* pos = nullptr;
    RowIndex index;
    hipError_t e = ids_bytes == 8 ? sort_positions<int64_t>((const int64_t*)ids, N, (int)V, by_bucket, L, ws, &keys, &pos, &index, stream)
                                  : sort_positions<int32_t>((const int32_t*)ids, N, (int)V, by_bucket, L, ws, &keys, &pos, &index, stream);
    if (e != hipSuccess) return e;
    const int* row_start = (const int*)(ws + L.row_start);
    float* partial = (float*)(ws + L.partial);
    auto rows = [&](auto zero, auto align) {
        typedef decltype(zero) TIn;
        return launch_rows_want<TIn, decltype(align)::value>(want, (const TIn*)G, row_start, keys, pos, N, (int)V, (int)T, d, index, partial, S_id, S_sq,
                                                             S_sign, stream);
    };
    constexpr std::integral_constant<int, 4> A4{};
    constexpr std::integral_constant<int, 2> A2{};
    constexpr std::integral_constant<int, 1> A1{};
    constexpr std::integral_constant<int, 0> A0{};
    if (dt == PEX_BF16) return d < CH ? rows(uint16_t{}, A0) : d % 4 == 0 ? rows(uint16_t{}, A4) : d % 2 == 0 ? rows(uint16_t{}, A2) : rows(uint16_t{}, A1);
    return d < CH ? rows(float{}, A0) : d % 4 == 0 ? rows(float{}, A4) : rows(float{}, A1);
}

}  // namespace pex
