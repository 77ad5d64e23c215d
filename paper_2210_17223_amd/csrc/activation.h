// Activations of the 16-bit layers and their derivatives, as the epilogues of the forward's and the
// backward's GEMMs evaluate them in fp32: a few per cent of the rounding that follows, and few issue
// slots -- a compute unit whose four wavefronts hold a 256 x 256 tile has nothing else to run beside its
// epilogue (first expert GEMM of 64 x 1024 rows, N = 8192, K = 2048, after thirty launches, one tile per block: 1845 us, 1729
// without the GeLU; 1860 with the form of two transcendentals).
#pragma once

#include <hip/hip_runtime.h>

namespace moe {

// GeLU(v) = max(v, 0) - a Phi(-a) with a = |v|, and Phi(-a) = 2^P(a), P a polynomial of degree 5
// fitted to log2 of the normal CDF (minimax of the error of a Phi(-a) on [0, 8] with P(0) = -1, so that small
// arguments are halved exactly and the error falls with v; the first coefficient sends it to zero beyond).
// Absolute error below 7.2e-7 with the rounding of results around 4, and below |v| (4e-5 |v| + 3e-7) beside
// one rounding of the result.  One transcendental and eight plain instructions; 1 / (1 + 2^(v Q(v^2))) with a
// cubic Q, which it replaces, took two and eight and was off by 1.4e-5.  (The clamp keeps infinity off the
// product; NaN stays NaN.)
__device__ __forceinline__ float gelu_erf_fast(float v)
{
    const float a = __builtin_elementwise_minimum(__builtin_fabsf(v), 10.0f);
    float p = -4.881171587e-04f;
    p = __builtin_fmaf(p, a, 7.198805226e-03f);
    p = __builtin_fmaf(p, a, -5.214680287e-02f);
    p = __builtin_fmaf(p, a, -4.595957109e-01f);
    p = __builtin_fmaf(p, a, -1.151000576e+00f);
    p = __builtin_fmaf(p, a, -1.0f);
    return __builtin_fmaf(-a, __builtin_amdgcn_exp2f(p), __builtin_elementwise_maximum(v, 0.0f));
}

// GeLU'(v) = Phi(v) + v phi(v) = 1 - D(v) for v >= 0 and D(-v) else, with D(a) = Phi(-a) - a phi(a) =
// exp(-a^2 / 2) R(a), R a polynomial of degree 7 (minimax of the error of D on [0, 6.5]).
// Absolute error below 4.2e-6 (2.9e-5 with the two functions apart, and two more transcendentals).  With it
// and the packed conversion to bf16 the dP GEMM of 63622 rows, 2048 x 8192, took 2461 us instead of 2530; of 8192
// rows, 768 x 3072, 89.4 instead of 92.4 (with the pre-activations still fetched behind its loop).
__device__ __forceinline__ float gelu_erf_derivative_fast(float v)
{
    const float a = __builtin_fabsf(v);
    float r = -1.685900643e-04f;
    r = __builtin_fmaf(r, a, 2.319469815e-03f);
    r = __builtin_fmaf(r, a, -1.392536145e-02f);
    r = __builtin_fmaf(r, a, 4.994355515e-02f);
    r = __builtin_fmaf(r, a, -1.258302778e-01f);
    r = __builtin_fmaf(r, a, 2.479609698e-01f);
    r = __builtin_fmaf(r, a, -7.976624370e-01f);
    r = __builtin_fmaf(r, a, 4.999959767e-01f);
    const float d = r * __builtin_amdgcn_exp2f(-0.72134752044448171f * (v * v));
    return v < 0.0f ? d : 1.0f - d;
}

// 0.5 (1 + tanh u) with u = sqrt(2 / pi) (v + 0.044715 v^3), as 1 / (1 + e^-2u): two transcendental
// instructions instead of tanhf
__device__ __forceinline__ float half_one_plus_tanh(float v)
{
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(v * (-2.3022082f - 0.10294324f * v * v)));
}

}  // namespace moe
