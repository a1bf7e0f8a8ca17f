// pex_bf16.h -- device helpers on packed bf16 values.  Device code only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pex {
namespace {

// two bf16 values -> squares in fp32 -> two bf16 (round to nearest even, one packed conversion); zero stays zero
__device__ __forceinline__ uint32_t square_pair_rne(uint32_t packed)
{
    typedef __attribute__((ext_vector_type(2))) float float2_t;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
    const float lo = __uint_as_float(packed << 16), hi = __uint_as_float(packed & 0xffff0000u);
    const float2_t sq = {lo * lo, hi * hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(sq, bf16x2_t));
}

// two bf16 values -> their squares exactly, each as the sum of two bf16: a square has at most 16 significant bits, `hi` holds
// the upper half of its fp32 form, `lo` the remainder.  Truncated, not rounded: a finite square stays finite and no half is
// negative, so sums over products of halves are non-finite only where the products of `hi` say so.
__device__ __forceinline__ void square_pair_split(uint32_t packed, uint32_t& hi, uint32_t& lo)
{
    const float a = __uint_as_float(packed << 16), b = __uint_as_float(packed & 0xffff0000u);
    const float sa = a * a, sb = b * b;
    const uint32_t ha = __float_as_uint(sa) & 0xffff0000u, hb = __float_as_uint(sb) & 0xffff0000u;
    hi = (ha >> 16) | hb;
    // an infinite square has no remainder
    const float ra = __builtin_isinf(sa) ? 0.f : sa - __uint_as_float(ha), rb = __builtin_isinf(sb) ? 0.f : sb - __uint_as_float(hb);
    lo = (__float_as_uint(ra) >> 16) | (__float_as_uint(rb) & 0xffff0000u);
}

}  // namespace
}  // namespace pex
