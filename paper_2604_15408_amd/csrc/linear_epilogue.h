// What the linear kernels share behind their main loops: GELU and the conversion of 16 consecutive outputs
// (internal).
#pragma once

#include "common.h"
#include "mfma_lds.h"

namespace ragged {

// GELU(t) = t * Phi(t) = max(t, 0) - |t| * Phi(-|t|), with Phi(-a) = 2^P(a) for 0 <= a <= 10: P is the degree-6
// polynomial that minimises the largest absolute error of a * 2^P(a) (a linear program over 6000 points of
// [0, 9]; evaluated in fp32 the error of GELU is at most 9e-8, and nothing cancels in the negative tail).  Beyond 10
// the argument is clamped: the term is then |t| * 2^-75 at most, far below any result.
// 9 VALU + 1 transcendental operation per element; the epilogue of an MFMA kernel does not overlap its matrix work, so
// this count is what the activation costs (an erfc quotient with rcp and exp2 took 11 + 2 and was accurate to 2.1e-7).
__device__ __forceinline__ float gelu_erf(float t) {
    const float a = fminf(fabsf(t), 10.0f);
    float p = __builtin_fmaf(a, 3.3139058359665796e-05f, -0.0007696275133639574f);
    p = __builtin_fmaf(p, a, 0.008082140237092972f);
    p = __builtin_fmaf(p, a, -0.05341433733701706f);
    p = __builtin_fmaf(p, a, -0.45876961946487427f);
    p = __builtin_fmaf(p, a, -1.1512017250061035f);
    p = __builtin_fmaf(p, a, -0.9999932646751404f);
    return __builtin_fmaf(-a, __builtin_amdgcn_exp2f(p), __builtin_elementwise_maximum(t, 0.f));   // (keeps a NaN, as fmaxf does not)
}

__device__ __forceinline__ void unpack16(F16, const uint4& a, const uint4& b, float (&v)[16]) {
    const f16x8 lo = as_vec8<f16x8>(a), hi = as_vec8<f16x8>(b);
#pragma unroll
    for (int e = 0; e < 8; ++e) { v[e] = (float)lo[e]; v[8 + e] = (float)hi[e]; }
}
__device__ __forceinline__ void unpack16(BF16, const uint4& a, const uint4& b, float (&v)[16]) {
    const bf16x8 lo = as_vec8<bf16x8>(a), hi = as_vec8<bf16x8>(b);
#pragma unroll
    for (int e = 0; e < 8; ++e) { v[e] = (float)lo[e]; v[8 + e] = (float)hi[e]; }
}
__device__ __forceinline__ void pack16(F16, const float (&v)[16], uint4& a, uint4& b) {
    f16x8 lo, hi;
#pragma unroll
    for (int e = 0; e < 8; ++e) { lo[e] = (_Float16)v[e]; hi[e] = (_Float16)v[8 + e]; }
    a = __builtin_bit_cast(uint4, lo);
    b = __builtin_bit_cast(uint4, hi);
}
__device__ __forceinline__ void pack16(BF16, const float (&v)[16], uint4& a, uint4& b) {
    bf16x8 lo, hi;
#pragma unroll
    for (int e = 0; e < 8; ++e) { lo[e] = (__bf16)v[e]; hi[e] = (__bf16)v[8 + e]; }
    a = __builtin_bit_cast(uint4, lo);
    b = __builtin_bit_cast(uint4, hi);
}

// Eight consecutive outputs of one row <-> 16 bytes.
__device__ __forceinline__ void unpack8(F16, const uint4& a, float (&v)[8]) {
    const f16x8 h = as_vec8<f16x8>(a);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (float)h[e];
}
__device__ __forceinline__ void unpack8(BF16, const uint4& a, float (&v)[8]) {
    const bf16x8 h = as_vec8<bf16x8>(a);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (float)h[e];
}
__device__ __forceinline__ uint4 pack8(F16, const float (&v)[8]) {
    f16x8 h;
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = (_Float16)v[e];
    return __builtin_bit_cast(uint4, h);
}
__device__ __forceinline__ uint4 pack8(BF16, const float (&v)[8]) {
    bf16x8 h;
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = (__bf16)v[e];
    return __builtin_bit_cast(uint4, h);
}

}  // namespace ragged
