// pex_f32.h -- what the two fp32 contraction kernels share.  Device code only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pex {
namespace {

typedef __attribute__((ext_vector_type(4))) float float4_t;
typedef __attribute__((ext_vector_type(4))) unsigned int uint4_t;
typedef float4_t __attribute__((aligned(4))) float4_u;      // four floats at any float's address

constexpr int F_T = 64;                    // edge of a wave's tile
constexpr int F_CHUNK = 1024;              // rows after which a plain contraction is folded into its sum
constexpr uint32_t F_OUTSIDE = 0x80000000u; // lane offset beyond every descriptor (windows stay below 2^30 bytes)

// What one launch produces (bit set); none of the per-example ones: a plain contraction over all rows, written to out_id
constexpr int F_ID = 1, F_SQ = 2, F_SG = 4, F_SG8 = 8, F_IDW = 16, F_POW = 32, F_NORM = 64, F_TOKEN = 128;
constexpr int F_PLAIN = 0;

__device__ __forceinline__ float sign_of(float m) { return (float)((m > 0.f) - (m < 0.f)); }
// |m|^alpha, zero stays zero
__device__ __forceinline__ float power_of(float m, float alpha)
{
    return __builtin_amdgcn_exp2f(alpha * __builtin_amdgcn_logf(__builtin_fabsf(m)));
}

}  // namespace
}  // namespace pex
