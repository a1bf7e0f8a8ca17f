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

}  // namespace
}  // namespace pex
