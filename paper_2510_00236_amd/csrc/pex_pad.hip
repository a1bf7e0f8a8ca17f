// pex_pad.hip -- bf16 operands whose rows are not whole 16-byte chunks, copied to rows that are.
//
// The MFMA kernels bring their operands in as 16-byte chunks at 16-byte addresses (direct-to-LDS loads), which the rows of a
// layer of odd width do not have.  Copying such an operand once to rows of the next multiple of 8 (zero-filled: a zero
// feature adds zero rows or columns to M_b, which are not stored) costs one pass at HBM speed and brings every statistic
// onto those kernels.
//
// For the per-token square the copies hold the squares, each as a pair of bf16 that is exact (the SIMT kernel, which these
// layers came from, keeps the squares in fp32): first the upper halves of the whole operand, then the remainders.  The four
// products of the halves are contracted one after the other into partial sums; where those of the upper halves overflow or hold an
// infinity or a NaN, they alone are the result.  B=14 T=544 3776x1943: 1735 us on the SIMT
// kernel, 451 so.
//
// Bound by HBM: 2 bytes read and 2 written per element.  A lane makes one 16-byte chunk of the copy from five dwords at
// 4-byte addresses (a row may start in the middle of a dword: then the five are shifted by 16 bits into four), four chunks
// in flight per lane.  Measured: 16000 rows of 2049 and 3001 elements in 54 us (6.0 TB/s); the layer's phi = square 3401 us on
// the SIMT kernel, 279 us with the copies.  B=8 T=256 768 x 50257, identity + square: 4253 -> 351 us, 92 of them for the copy.
#include "pex_bf16.h"
#include "pex_internal.h"

namespace pex {
namespace {

typedef __attribute__((ext_vector_type(4))) unsigned int uint4_t;
typedef uint4_t __attribute__((aligned(4))) uint4_u;      // four dwords at any dword's address

constexpr int PAD_CHUNKS = 4;      // chunks per lane, 256 apart

// elements e0 .. e0+7 of `in` (of `total`), those from `count` on as zeros
__device__ __forceinline__ uint4_t load_chunk(const uint16_t* __restrict__ in, int64_t e0, int count, int64_t total)
{
    uint4_t v;
    if (e0 + 8 < total) {          // the fifth dword ends at or before the end of the operand
        const uint32_t* w = reinterpret_cast<const uint32_t*>(in) + (e0 >> 1);
        v = *(const uint4_u*)w;
        if (e0 & 1) {
            const uint32_t next = w[4];
            v = uint4_t{__builtin_amdgcn_alignbit(v[1], v[0], 16), __builtin_amdgcn_alignbit(v[2], v[1], 16),
                        __builtin_amdgcn_alignbit(v[3], v[2], 16), __builtin_amdgcn_alignbit(next, v[3], 16)};
        }
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const int keep = count - 2 * d;      // elements of this dword that belong to the row
            v[d] &= keep >= 2 ? 0xffffffffu : (keep == 1 ? 0xffffu : 0u);
        }
    } else {
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t lo = 2 * d < count ? in[e0 + 2 * d] : 0u, hi = 2 * d + 1 < count ? in[e0 + 2 * d + 1] : 0u;
            v[d] = lo | (hi << 16);
        }
    }
    return v;
}

struct PadOperand {
    const uint16_t* in;
    uint4_t* out;
    int width, chunks;      // elements per row, 16-byte chunks per row of the copy
};

template <bool SQUARES>
__global__ __launch_bounds__(256) void pad_rows_kernel(PadOperand a, PadOperand b, int64_t rows)
{
    const PadOperand o = blockIdx.y == 0 ? a : b;
    const uint32_t n = (uint32_t)(rows * o.chunks);          // below 2^31 (see pad_supports)
    const int64_t total = rows * o.width;
    const uint32_t first = blockIdx.x * (256 * PAD_CHUNKS) + threadIdx.x;
    uint4_t v[PAD_CHUNKS];
#pragma unroll
    for (int u = 0; u < PAD_CHUNKS; ++u) {
        const uint32_t k = first + 256 * u;
        if (k >= n) continue;
        const uint32_t row = k / (uint32_t)o.chunks, c = k - row * (uint32_t)o.chunks;
        v[u] = load_chunk(o.in, (int64_t)row * o.width + 8 * c, o.width - (int)(8 * c), total);
    }
#pragma unroll
    for (int u = 0; u < PAD_CHUNKS; ++u) {
        const uint32_t k = first + 256 * u;
        if (k >= n) continue;
        if constexpr (SQUARES) {
            uint4_t hi, lo;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t h, l;
                square_pair_split(v[u][d], h, l);
                hi[d] = h;
                lo[d] = l;
            }
            o.out[k] = hi;
            o.out[(int64_t)n + k] = lo;
        } else o.out[k] = v[u];
    }
}

}  // namespace

int64_t padded_width(int64_t width) { return (width + 7) / 8 * 8; }

bool pad_supports(int64_t rows, int64_t din, int64_t dout)
{
    const int64_t lim = (int64_t)1 << 31;
    return din < lim / 2 && dout < lim / 2 && rows * (padded_width(din) / 8) < lim && rows * (padded_width(dout) / 8) < lim;
}

hipError_t launch_pad_rows(const void* X, void* x_out, const void* G, void* g_out, int64_t rows, int64_t din, int64_t dout, bool squares,
                           hipStream_t stream)
{
    PadOperand op[2];
    int count = 0;
    int64_t most = 0;
    auto add = [&](const void* in, void* out, int64_t width) {
        if (!out) return;
        op[count] = PadOperand{(const uint16_t*)in, (uint4_t*)out, (int)width, (int)(padded_width(width) / 8)};
        if (rows * op[count].chunks > most) most = rows * op[count].chunks;
        ++count;
    };
    add(X, x_out, din);
    add(G, g_out, dout);
    if (count == 0) return hipSuccess;
    if (count == 1) op[1] = op[0];
    const dim3 grid((unsigned)((most + 256 * PAD_CHUNKS - 1) / (256 * PAD_CHUNKS)), (unsigned)count), block(256);
    if (squares) pad_rows_kernel<true><<<grid, block, 0, stream>>>(op[0], op[1], rows);
    else pad_rows_kernel<false><<<grid, block, 0, stream>>>(op[0], op[1], rows);
    return hipGetLastError();
}

}  // namespace pex
