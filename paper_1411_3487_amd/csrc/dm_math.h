// dm_math.h -- FP64 elementary functions of the step kernels (device only),
// for the arguments those kernels have.
//
// The hardware's v_rsq_f64 / v_rcp_f64 seeds (relative error below 2^-25) are
// refined by Newton and Goldschmidt steps, and the logarithm, sine and cosine
// of Box-Muller use polynomials interpolated at the Chebyshev nodes of their
// reduced range.  No argument is denormal, none needs a large-argument
// reduction, and the angle is reduced exactly in integers, which is what the
// general library functions spend most of their instructions on.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dm {

#if defined(__HIP_DEVICE_COMPILE__) || defined(__HIPCC__)

__device__ __forceinline__ double fma64(double a, double b, double c)
{
    return __builtin_fma(a, b, c);
}

// 1 / sqrt(x) for normal x > 0 (x = 0 or Inf gives NaN): one third-order
// step y (1 + e/2 + 3 e^2 / 8) with e = 1 - x y^2.
__device__ __forceinline__ double rsqrt64(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma64(-(x * y), y, 1.0);
    return fma64(y * e, fma64(e, 0.375, 0.5), y);
}

// sqrt(x) for normal x > 0 (x = 0 gives NaN): Goldschmidt's coupled step for
// sqrt(x) and 1/(2 sqrt(x)), then the residual x - g^2 once.
__device__ __forceinline__ double sqrt64(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma64(-h, g, 0.5);
    g = fma64(g, r, g);
    h = fma64(h, r, h);
    return fma64(fma64(-g, g, x), h, g);
}

// a / b for normal b: the refined reciprocal, then the residual once.
__device__ __forceinline__ double div64(double a, double b)
{
    double y = __builtin_amdgcn_rcp(b);
    y = fma64(fma64(-b, y, 1.0), y, y);
    const double q = a * y;
    return fma64(fma64(-b, q, a), y, q);
}

// -2 ln u of u = (x + 1/2) 2^-32, x any 32-bit word: u = 2^k m with m in
// [sqrt(1/2), sqrt(2)) (so k = 0 next to u = 1 and nothing cancels),
// ln m = 2 atanh(s) = 2 s + s^3 P(s^2), s = (m - 1) / (m + 1).
__device__ __forceinline__ double neg2log_u32(uint32_t x)
{
    const double y = (double)x + 0.5;
    const uint64_t b = __builtin_bit_cast(uint64_t, y);
    const int hi = (int)(b >> 32);
    const int k = (hi - 0x3fe6a09e) >> 20;  // high word of sqrt(1/2)
    const double m = __builtin_bit_cast(
        double, ((uint64_t)(uint32_t)(hi - (k << 20)) << 32) | (uint32_t)b);
    const double s = div64(m - 1.0, m + 1.0);
    const double z = s * s;
    // -2 P, degree 6 on [0, ((sqrt(2) - 1) / (sqrt(2) + 1))^2]
    double p = -2.0 * 0.14616585424934123;
    p = fma64(p, z, -2.0 * 0.1533171061820642);
    p = fma64(p, z, -2.0 * 0.18182889455675105);
    p = fma64(p, z, -2.0 * 0.22222211130259875);
    p = fma64(p, z, -2.0 * 0.2857142862600327);
    p = fma64(p, z, -2.0 * 0.39999999999899444);
    p = fma64(p, z, -2.0 * 0.666666666666667);
    const double w = fma64(p, z, -4.0);
    return fma64(w, s, (double)(k - 32) * -1.3862943611198906);  // -2 ln 2
}

// cos and sin of 2 pi (x + 1/2) 2^-32: the angle is (q + r) quarter turns
// with r in (-1/2, 1/2) exactly.
__device__ __forceinline__ void sincos_u32(uint32_t x, double &c, double &s)
{
    const uint32_t t = x + 0x20000000u;  // quadrant in the top two bits
    const double r = fma64((double)((int)(x << 2) >> 2), 0x1p-30, 0x1p-31);
    const double z = r * r;
    double a = 5.633933781537854e-08;  // sin(pi r / 2) / r in r^2
    a = fma64(a, z, -3.59864335298231e-06);
    a = fma64(a, z, 0.0001604411507421909);
    a = fma64(a, z, -0.004681754132340976);
    a = fma64(a, z, 0.07969262624604301);
    a = fma64(a, z, -0.6459640975062443);
    a = fma64(a, z, 1.5707963267948966);
    a *= r;
    double b = -6.329396344967424e-09;  // (cos(pi r / 2) - 1) / r^2 in r^2
    b = fma64(b, z, 4.710678405505227e-07);
    b = fma64(b, z, -2.5202039028029178e-05);
    b = fma64(b, z, 0.0009192602745468447);
    b = fma64(b, z, -0.020863480763340773);
    b = fma64(b, z, 0.2536695079010478);
    b = fma64(b, z, -1.2337005501361697);
    b = fma64(b, z, 1.0);
    const bool odd = (t & 0x40000000u) != 0;
    const uint64_t sc = (uint64_t)((t + 0x40000000u) & 0x80000000u) << 32;
    const uint64_t ss = (uint64_t)(t & 0x80000000u) << 32;
    c = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, odd ? a : b) ^ sc);
    s = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, odd ? b : a) ^ ss);
}

#endif

}  // namespace dm
