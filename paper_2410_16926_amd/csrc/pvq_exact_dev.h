// Correctly rounded float32 quotients and roots in a few instructions, for arguments between bounds.  What the compiler makes of
// / and sqrtf serves every argument and takes ten to eighteen; the results here are the same bits where the bounds hold, and
// the callers look (mostly a wave at a time) and take the general operations where they do not.
#pragma once

#include <hip/hip_runtime.h>

namespace pvq_exact_dev {

// lo <= |x| < hi
__device__ inline bool magnitude_in(float x, float lo, float hi)
{
    const uint32_t l = 2u * __float_as_uint(lo), h = 2u * __float_as_uint(hi);
    return 2u * __float_as_uint(x) - l < h - l;
}

// RN(1 / b): v_rcp_f32 and one step of Newton's.  Every significand has been compared with the division; b from 2^-100 to 2^100.
__device__ inline float reciprocal(float b)
{
    const float y = __builtin_amdgcn_rcpf(b);
    return __builtin_fmaf(__builtin_fmaf(-b, y, 1.0f), y, y);
}

// A divisor b with its reciprocal y = RN(1 / b) and what that is off by, yl = y (1 - b y).  The first quotient a y + a yl is the
// exact one to a few parts in 2^47, so rounded it is one of the two floats next to it; then a - q b is exact, and
// q + (a - q b) y rounds to RN(a / b) (Markstein, Computation of elementary functions on the IBM RISC System/6000 processor,
// 1990).  |b| from 2^-60 to 2^60, |a| from 2^-90 to 2^90 and |a / b| from 2^-100 to 2^100, where nothing over- or underflows (a = +0
// gives +0 too if b > 0; -0 does not keep its sign).
struct divisor { float b, y, yl; };
__device__ inline divisor divisor_of(float b, float y)
{
    divisor d;
    d.b = b;
    d.y = y;
    d.yl = __builtin_fmaf(-b, y, 1.0f) * y;
    return d;
}
__device__ inline float divide(float a, const divisor &d)
{
    const float q = __builtin_fmaf(a, d.y, a * d.yl);
    return __builtin_fmaf(__builtin_fmaf(-q, d.b, a), d.y, q);
}

// RN(k / l) for an integer 1 <= k <= 255 and l from 2^-100 to 2^100: the first quotient with v_rcp_f32 and one correction.  Every k
// with every significand of l has been compared with the division (the first that differs is 367).
__device__ inline float small_over(float k, float l)
{
    const float y = __builtin_amdgcn_rcpf(l), q = k * y;
    return __builtin_fmaf(__builtin_fmaf(-q, l, k), y, q);
}
// The same for integers up to 1023, with the reciprocal's own step (every k and significand compared likewise).
__device__ inline float integer_over(float k, float l)
{
    const float y = reciprocal(l), q = k * y;
    return __builtin_fmaf(__builtin_fmaf(-q, l, k), y, q);
}

// RN(sqrt(x)), x from 2^-100 to 2^100, y0 = v_rsq_f32 of x: every float of them compared with sqrtf.
__device__ inline float root_of(float x, float y0)
{
    const float g = x * y0, h = 0.5f * y0;
    return __builtin_fmaf(__builtin_fmaf(-g, g, x), h, g);
}
__device__ inline float root_of(float x) { return root_of(x, __builtin_amdgcn_rsqf(x)); }

// The root of an integer 1 <= n <= 2^16 as a divisor (its reciprocal from the same v_rsq_f32 and one step: RN for all of them).
__device__ inline divisor root_divisor(float n)
{
    const float y0 = __builtin_amdgcn_rsqf(n), root = root_of(n, y0);
    return divisor_of(root, __builtin_fmaf(__builtin_fmaf(-root, y0, 1.0f), y0, y0));
}

}  // namespace pvq_exact_dev
