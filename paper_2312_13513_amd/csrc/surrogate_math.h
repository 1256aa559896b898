// Device arithmetic shared by the surrogate's kernels: BF16 conversions, the
// GELU and its derivative, MFMA operand types.
#pragma once

#include "surrogate.h"

namespace chem {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// FP32 -> BF16, round to nearest, ties to even; NaN -> quiet NaN.
__device__ __forceinline__ bf16_t to_bf16(float f)
{
    unsigned u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)0x7fc0;
    u += 0x7fffu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

// GELU(u) = u Phi(u) without branches: Phi(-|u|) = erfc(z)/2, z = |u|/sqrt(2),
// in the form erfc(z) = t exp(-z^2 + P(t)), t = 1/(1 + z/2) (Numerical
// Recipes' erfcc), P of degree 7 refitted in FP64 (gelu_fit.py).  Evaluated
// through the hardware base-2 exponential with 1/2 and log2(e) folded into
// the coefficients, Phi(-|u|) = t 2^(Q(t) - u^2 log2(e)/2), Q = log2(e) P - 1,
// and GELU(u) = max(u, 0) - |u| Phi(-|u|) (one fused multiply-add for both
// signs; an infinite u gives NaN there).  Relative error within 1.7e-5 of
// the exact GELU for every finite u; the activations are then rounded to
// BF16 (unit roundoff 2^-8).
__device__ __forceinline__ float gelu(float u)
{
    const float a = fabsf(u);
    const float t = __builtin_amdgcn_rcpf(fmaf(a, 0.35355339059327373f, 1.0f));
    float q = -2.396635413e-01f;
    q = fmaf(q, t, 9.644635320e-01f);
    q = fmaf(q, t, -1.259334445e+00f);
    q = fmaf(q, t, 3.582076728e-01f);
    q = fmaf(q, t, 5.822304171e-03f);
    q = fmaf(q, t, 5.541245341e-01f);
    q = fmaf(q, t, 1.442124605e+00f);
    q = fmaf(q, t, -2.825743914e+00f);
    const float half = t * __builtin_amdgcn_exp2f(fmaf(u * u, -0.72134752044448170f, q));
    return fmaf(-a, half, fmaxf(u, 0.0f));
}

// Activation FP32 -> BF16 with the hardware conversion (round to nearest even).
__device__ __forceinline__ bf16_t act_bf16(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }

__device__ __forceinline__ float gelu_grad(float u)
{
    return 0.5f * (1.0f + erff(u * 0.70710678118654752f)) +
           u * expf(-0.5f * u * u) * 0.39894228040143268f;
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace chem
