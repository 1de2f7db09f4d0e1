// The activations, element by element: shared by the row-wise kernels and by the epilogues that apply them to a GEMM's result.
#pragma once
#include <hip/hip_runtime.h>

namespace ob {
namespace {

// GELU through h = Phi(-|z|) = erfc(|z| / sqrt 2) / 2 = t Q(t) e^(-z^2 / 2), t = 1 / (1 + 0.43 |z| / sqrt 2), Q the degree-7
// polynomial that is closest in the relative sense to erfc(x) e^(x^2) / t over x <= 9.5 (a Lawson fit to 8000 Chebyshev
// nodes; 1.5e-7 with its coefficients in fp32): an exponential, a reciprocal and 8 FMAs, where erff() takes twice that and
// 1 + erf(z) cancels for negative z.  Over bf16 arguments h is within 8.2e-7 of its value for |z| <= 4, 2.2e-6 to 6 and 1.2e-5
// to 13 (the rounding of z^2 in the exponent), relative; so is GELU.  The derivative takes h as it is for negative z too
// (0.5 - (0.5 - h) cancels: 3 % at z = -6) and the same exponential for the density: within 1.2e-5 for z <= -1,
// 7e-8 absolute around its zero at -0.75.  (These kernels were bound by the vector unit, not by HBM.)
struct HalfTail { float h, e; };   // Phi(-|z|), e^(-z^2 / 2)
__device__ __forceinline__ HalfTail half_tail(float z) {
    const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(fabsf(z), 0.30405592f, 1.0f));
    const float y = z * 0.84932180f;             // e^(-z^2 / 2) = 2^(-y^2)
    const float e = __builtin_amdgcn_exp2f(-y * y);
    float q = 0.036854025f;
    q = __builtin_fmaf(q, t, -0.15518695f);
    q = __builtin_fmaf(q, t, 0.19185331f);
    q = __builtin_fmaf(q, t, -0.042863335f);
    q = __builtin_fmaf(q, t, 0.12342247f);
    q = __builtin_fmaf(q, t, 0.10247547f);
    q = __builtin_fmaf(q, t, 0.12218773f);
    q = __builtin_fmaf(q, t, 0.12125731f);
    return HalfTail{q * t * e, e};
}
__device__ __forceinline__ float gelu_f(float z) {
    const float h = half_tail(z).h;
    return z * (z < 0.0f ? h : 1.0f - h);
}
__device__ __forceinline__ float gelu_grad_f(float z) {
    const HalfTail k = half_tail(z);
    return __builtin_fmaf(z * k.e, 0.3989422804014327f, z < 0.0f ? k.h : 1.0f - k.h);
}
__device__ __forceinline__ float sigmoid_f(float z) { return 1.0f / (1.0f + __expf(-z)); }
// gradients of silu(gate) * up, d that of the product
struct SwigluGrad { float gate, up; };
__device__ __forceinline__ SwigluGrad swiglu_grad_f(float d, float gate, float up) {
    const float sg = sigmoid_f(gate);
    return SwigluGrad{d * up * sg * (1.0f + gate * (1.0f - sg)), d * gate * sg};
}

}  // namespace
}  // namespace ob
