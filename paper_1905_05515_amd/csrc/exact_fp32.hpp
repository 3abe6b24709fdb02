// Correctly rounded binary32 reciprocal, square root and quotient for
// operands of a known range, as short sequences around the hardware's
// approximations (v_rcp_f32, v_rsq_f32: within 1 ulp).  The general
// operators must also serve denormals, infinities and zeros and cost 11
// (division) and 14 (square root) instructions each; in the Kalman step of
// one track, a serial chain that a wave issues at one instruction per four
// cycles, they made up 95 of the transport's 168 instructions (now 115 with
// the gain's reciprocal).  One sector's tracking 592 -> 520 us, a central
// event's 678 -> 629 us, its merge and full-track fit 1053 -> 933 us; the
// 512-instance step, bound by memory latency, unchanged at 3738 us.
//
// Method: Newton steps with fused multiply-adds, whose residuals are exact
// (Markstein, IBM J. Res. Dev. 34, 1990: a correctly rounded reciprocal y of
// b and a faithful quotient q give RN(q + RN(a - b q) y) = RN(a / b)).  That
// the one-step reciprocal and square root are the correctly rounded ones on
// their whole range is checked over every float of it by
// tests/test_gpu_exact_fp32.py.
#pragma once
#include <hip/hip_runtime.h>

#pragma clang fp contract(off)

namespace tpc {

// 1 / b for kRcpMin <= |b| <= kRcpMax
constexpr float kRcpMin = 0x1p-125f, kRcpMax = 0x1p125f;

__device__ __forceinline__ float rcp_exact(float b)
{
    const float r = __builtin_amdgcn_rcpf(b);
    return fmaf(fmaf(-b, r, 1.0f), r, r);
}

// 1 / b for any b: the short form unless a lane of the wave is outside its
// range (a branch the whole wave skips; as a select both would be computed)
__device__ __forceinline__ float rcp_any(float b)
{
    const bool in = fabsf(b) >= kRcpMin && fabsf(b) <= kRcpMax;
    float r = rcp_exact(b);
    if (__builtin_expect(__ballot(!in) != 0ull, 0)) r = 1.0f / b;
    return r;
}

// sqrt(u) for 2^-100 <= u <= 2^120
__device__ __forceinline__ float sqrt_exact(float u)
{
    const float y = __builtin_amdgcn_rsqf(u);
    const float g = u * y;
    return fmaf(fmaf(-g, g, u), 0.5f * y, g);
}

// a / b given r = rcp_exact(b) (not an approximation an ulp off: for a b of
// all ones, 1 - 2^-24 say, the last step rounds right only with it);
// kDivMin <= |b| <= kDivMax and a zero or 2^-80 <= |a| <= 2^80 (a smaller |a|
// gives a quotient below 2^-60 that may be off; the quotient of a negative
// zero is a positive zero)
constexpr float kDivMin = 0x1p-20f, kDivMax = 0x1p20f;

__device__ __forceinline__ float div_exact(float a, float b, float r)
{
    float q = a * r;
    q = fmaf(fmaf(-b, q, a), r, q);       // within an ulp
    return fmaf(fmaf(-b, q, a), r, q);
}

// the same, and the operator's result for zeros of either sign, infinities
// and NaN in a
__device__ __forceinline__ float div_exact_special(float a, float b, float r)
{
    return __builtin_amdgcn_div_fixupf(div_exact(a, b, r), b, a);
}

}  // namespace tpc
