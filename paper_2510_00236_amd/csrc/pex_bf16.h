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

// two bf16 values -> their squares exactly, each as the sum of two bf16: a square has at most 16 significant bits, `hi` is
// rounded to nearest, the remainder fits the 8 bits of `lo`
__device__ __forceinline__ void square_pair_split(uint32_t packed, uint32_t& hi, uint32_t& lo)
{
    typedef __attribute__((ext_vector_type(2))) float float2_t;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
    const float a = __uint_as_float(packed << 16), b = __uint_as_float(packed & 0xffff0000u);
    hi = square_pair_rne(packed);
    const float ha = __uint_as_float(hi << 16), hb = __uint_as_float(hi & 0xffff0000u);
    // a square beyond bf16's range has no remainder
    const float2_t rest = {__builtin_isinf(ha) ? 0.f : fmaf(a, a, -ha), __builtin_isinf(hb) ? 0.f : fmaf(b, b, -hb)};
    lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(rest, bf16x2_t));
}

}  // namespace
}  // namespace pex
