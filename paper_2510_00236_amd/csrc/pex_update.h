// pex_update.h -- the arithmetic of the optimizer updates and of the moment tracking, shared by the kernels that do one tensor
// and those that do a whole model's.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "pex.h"

namespace pex {
namespace {

// 16-byte accesses, past the caches where STREAM: a tensor whose buffers exceed the memory-side cache evicts itself on every
// pass (see `streams`)
template <bool STREAM>
__device__ __forceinline__ float4 load4(const float4* p)
{
    typedef __attribute__((ext_vector_type(4))) float f4;
    if constexpr (STREAM) {
        const f4 q = __builtin_nontemporal_load((const f4*)p);
        return make_float4(q[0], q[1], q[2], q[3]);
    } else return *p;
}
template <bool STREAM>
__device__ __forceinline__ void store4(float4* p, const float4& v)
{
    typedef __attribute__((ext_vector_type(4))) float f4;
    if constexpr (STREAM) __builtin_nontemporal_store(f4{v.x, v.y, v.z, v.w}, (f4*)p);
    else *p = v;
}

struct AdamConsts {
    float beta1, one_m_beta1, beta2, one_m_beta2;
    float inv_bc1, inv_bc2;   // 1/(1-beta1^t), 1/(1-beta2^t)
    float eps, eps_root, lr, wd, gs, qs;
    float c_est, inv_B;       // 1/(1-1/B), 1/B
};

template <int VARIANT>
__device__ __forceinline__ void adam_one(float& th, float& m, float& v, float sid, float ssq, const AdamConsts& k)
{
    const float mu_t = k.gs * sid;
    const float nu_adam = mu_t * mu_t;
    float nu_t;
    if (VARIANT == PEX_ADAM) nu_t = nu_adam;
    else {
        const float nu_micro = k.qs * ssq;
        if (VARIANT == PEX_MICROADAM) nu_t = nu_micro;
        else if (VARIANT == PEX_MICROADAM_VAR) nu_t = k.c_est * (nu_micro - nu_adam);
        else nu_t = k.c_est * (nu_adam - nu_micro * k.inv_B);
    }
    m = fmaf(k.beta1, m, k.one_m_beta1 * mu_t);
    v = fmaf(k.beta2, v, k.one_m_beta2 * nu_t);
    const float mh = m * k.inv_bc1;
    float vh = v * k.inv_bc2;
    if (VARIANT == PEX_MICROADAM_VAR || VARIANT == PEX_MICROADAM_MSQ) vh = fmaxf(0.f, vh);
    const float u = mh / (sqrtf(vh + k.eps_root) + k.eps);
    th = th - k.lr * u - k.wd * th;
}

// every per-example gradient times kappa = min(1, max_norm / norm of the mean gradient)
__device__ __forceinline__ void clip(AdamConsts& k, double sum_sq, float max_norm)
{
    const double norm = fabs((double)k.gs) * sqrt(sum_sq);
    const float kappa = norm > (double)max_norm ? (float)((double)max_norm / norm) : 1.0f;
    k.gs *= kappa;
    k.qs *= kappa * kappa;
}

struct MomentConsts {
    float beta2, one_m_beta2, gs, qs;
    double corr, c_est, inv_B;   // 1/(1-beta2^t) or 1, 1/(1-1/B), 1/B
};

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// the two EMAs of one parameter, its estimates added to the sums
__device__ __forceinline__ void moment_one(float& a, float& q, float sid, float ssq, const MomentConsts& k, double& sum_mu2, double& sum_sigma2)
{
    const float mu_t = k.gs * sid;
    a = fmaf(k.beta2, a, k.one_m_beta2 * (mu_t * mu_t));
    q = fmaf(k.beta2, q, k.one_m_beta2 * (k.qs * ssq));
    const double ah = (double)a * k.corr, qh = (double)q * k.corr;
    sum_mu2 += k.c_est * (ah - qh * k.inv_B);
    sum_sigma2 += k.c_est * (qh - ah);
}

inline AdamConsts adam_consts(const pex_adam_params& p)
{
    AdamConsts k;
    k.beta1 = p.beta1; k.one_m_beta1 = 1.f - p.beta1;
    k.beta2 = p.beta2; k.one_m_beta2 = 1.f - p.beta2;
    k.inv_bc1 = (float)(1.0 / (1.0 - pow((double)p.beta1, (double)p.step)));
    k.inv_bc2 = (float)(1.0 / (1.0 - pow((double)p.beta2, (double)p.step)));
    k.eps = p.eps; k.eps_root = p.eps_root; k.lr = p.lr; k.wd = p.weight_decay;
    k.gs = p.grad_scale; k.qs = p.sq_scale;
    k.inv_B = 1.f / (float)p.B;
    k.c_est = p.B > 1 ? (float)(1.0 / (1.0 - 1.0 / (double)p.B)) : 0.f;
    return k;
}

inline MomentConsts moment_consts(const pex_moment_params& p)
{
    MomentConsts k;
    k.beta2 = p.beta2; k.one_m_beta2 = 1.f - p.beta2;
    k.gs = p.grad_scale; k.qs = p.sq_scale;
    k.corr = p.debias ? 1.0 / (1.0 - pow((double)p.beta2, (double)p.step)) : 1.0;
    k.inv_B = 1.0 / (double)p.B;
    k.c_est = 1.0 / (1.0 - k.inv_B);
    return k;
}

// Buffers of n floats that together exceed the 256 MB memory-side cache by so much that a pass evicts what the next one would have
// found are accessed past the caches.  Measured on repeated passes (cached / streamed, us), Adam family on five buffers: 320 MiB
// 84 / 93, 340 91 / 96, 360 104 / 104, 380 114 / 108, 500 159 / 144; on four buffers 360 118 / 113; sign updates 340 100 / 99; moment
// tracking 340 86 / 92, 360 98 / 98, 400 117 / 108.
inline bool streams(int64_t n, int buffers) { return n * buffers * 4 > (int64_t)360 << 20; }

}  // namespace
}  // namespace pex
