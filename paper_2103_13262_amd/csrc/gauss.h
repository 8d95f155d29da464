// The Gaussian factors of GeLU and of its derivative, evaluated directly (internal; compiled for the host as well).
//
// For a = |z| the scaled complement m = exp(a^2 / 2) Phi(-a) falls smoothly from 1/2 to 0; mapped to a finite interval, s = 0.3 a / (1 + 0.3 a),
// one polynomial covers all of it (the method of Shepherd and Laframboise, "Chebyshev approximation of (1 + 2x) exp(x^2) erfc x in
// 0 <= x < infinity", Math. Comp. 36, 1981).  The nine coefficients are a weighted least-squares fit of (m - 1/2) / s for a up to 14, from
// 64-bit values of the scaled complement; m = 1/2 + s R(s) keeps the absolute error at the last bit where z is small, the factor exp(-a^2 / 2)
// keeps the relative one where it is large and negative.  In 32 bits: Phi(z) off by less than 1e-5 of itself for all z above -9 and by less than
// 1.3e-7; the derivative by less than 1.3e-7.  The table of the persistent kernels (ggemm_bf16_sk.h) is off by 1e-7 inside its
// range and by up to 4e-4 outside, and its H, carried from the rounded z to z along the slope, by up to 6e-3 of itself at z = -7.
// (Five coefficients, Abramowitz and Stegun 7.1.26, are off by 0.4 % of Phi at z = -6 and 1 % at -8, and by 4e-7 in the derivative; they
// made a pass 0.2 to 1 % shorter: 2048 tokens, 64 experts, d 1024, h 2048: 464 us, with these 469; 8 tokens, 16 experts, d 1024, h 4096: 53.8, 54.2.)
#pragma once
#include <math.h>

#if defined(__HIPCC__)
#define MOE_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define MOE_HOST_DEVICE inline
#endif

namespace moe {

struct Tail { float a, e, m; };     // |z| (at most 16), exp(-a^2 / 2), exp(a^2 / 2) Phi(-a)

MOE_HOST_DEVICE Tail normal_tail(float z)
{
    Tail r;
    r.a = fabsf(z) > 16.f ? 16.f : fabsf(z);      // (beyond 16 Phi is 0 or 1, and an infinite z must not meet a zero; a NaN stays one)
    const float x = r.a * r.a * -0.72134752044448170f;      // (-log2(e) / 2)
#if defined(__HIP_DEVICE_COMPILE__)
    const float t = __builtin_amdgcn_rcpf(fmaf(r.a, 0.3f, 1.0f));
    r.e = __builtin_amdgcn_exp2f(x);
#else
    const float t = 1.0f / fmaf(r.a, 0.3f, 1.0f);
    r.e = exp2f(x);
#endif
    const float s = r.a * 0.3f * t;
    float p = 0.0076907324f;
    p = fmaf(s, p, 0.008930582f);
    p = fmaf(s, p, -0.0905263f);
    p = fmaf(s, p, 0.0776775f);
    p = fmaf(s, p, 0.12921643f);
    p = fmaf(s, p, -0.051005658f);
    p = fmaf(s, p, -0.7001714f);
    p = fmaf(s, p, 1.4480183f);
    p = fmaf(s, p, -1.3298087f);
    r.m = fmaf(s, p, 0.5f);
    return r;
}

// Phi(z)
MOE_HOST_DEVICE float normal_cdf(float z)
{
    const Tail t = normal_tail(z);
    const float q = t.m * t.e;
    return z < 0.f ? q : 1.0f - q;
}

// Phi(z) + z phi(z): the derivative of GeLU(z) = z Phi(z).  (At -z it is 1 minus what it is at z.)
MOE_HOST_DEVICE float gelu_slope(float z)
{
    const Tail t = normal_tail(z);
    const float q = t.e * fmaf(t.a, -0.39894228040143268f, t.m);
    return z < 0.f ? q : 1.0f - q;
}

}  // namespace moe
