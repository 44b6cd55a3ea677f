// Device helpers shared by the stencil kernels: a full-precision reciprocal, the fifth-order WENO
// derivative of Sec. 3.1 (Jiang-Peng form with the Jiang-Shu smoothness indicators) and the
// regularised Heaviside of the two-phase mixture.
#pragma once

#include <hip/hip_runtime.h>

namespace evp {

// reciprocal to full precision.  FP64: the hardware estimate (measured |1 - a x| <= 2^-24.4 over
// 2^-300 .. 2^300) refined by one third-order step, x <- x (1 + e + e^2), e = 1 - a x: 2^-53, as two
// Newton steps give, with one operation less.  FP32: one Newton step (x <- x (2 - a x)).
__device__ __forceinline__ double fast_rcp(double a)
{
    double x = __builtin_amdgcn_rcp(a);
    const double e = fma(-a, x, 1.0);
    return fma(x, fma(e, e, e), x);
}
__device__ __forceinline__ float fast_rcp(float a)
{
    float x = __builtin_amdgcn_rcpf(a);
    return fmaf(x, fmaf(-a, x, 1.0f), x);
}
// reciprocal square root of a >= 0, the argument limited to 2^-1000 .. 2^1000 and 2^-120 .. 2^120 (so that
// 0 and infinity give finite results): the hardware estimate refined by one step x <- x + x e / 2 (+ 3 x e^2 / 8 in
// FP64), e = 1 - a x^2.  1 - t fast_rsqrt(a) over a = t^2 .. 10^12 t^2 is off by at most 1.2e-16 and
// 6.6e-8 (1 - t / sqrt(a): 1.4e-16 and 7.5e-8) and takes a third of the instructions.
__device__ __forceinline__ double fast_rsqrt(double a)
{
    a = fmin(fmax(a, 0x1p-1000), 0x1p1000);
    const double x = __builtin_amdgcn_rsq(a);
    const double e = fma(-a * x, x, 1.0);
    return fma(x * e, fma(0.375, e, 0.5), x);
}
__device__ __forceinline__ float fast_rsqrt(float a)
{
    a = fminf(fmaxf(a, 0x1p-120f), 0x1p120f);
    const float x = __builtin_amdgcn_rsqf(a);
    const float e = fmaf(-a * x, x, 1.0f);
    return fmaf(0.5f * x, e, x);
}

// Fifth-order WENO from the five undivided one-sided differences v1..v5 (spacing folded out):
// returns h * dB/dx.  eps2 = eps h^2 keeps the weights equal to those of the divided form.
// Written on the differences s_k = v_{k+1} - v_k: the three candidate stencils are v3 plus
// q1 = -s1/3 + 5 s2/6, q2 = s2/6 + s3/3, q3 = 2 s3/3 - s4/6, and the Jiang-Shu indicators are
// 13/12 a_k^2 + 1/4 b_k^2 with a_k = s_{k+1} - s_k and b = 3 s2 - s1, s2 + s3, s4 - 3 s3 (the
// same numbers as the usual form in v, up to the sign of b).  The weights d_k / (eps + IS_k)^2,
// normalised, are invariant under a common scale of the indicators, so they are formed from
// 4 (eps + IS_k) = 4 eps + 13/3 a_k^2 + b_k^2, and over the common denominator
// e1^2 e2^2 e3^2: w_k = d_k prod_{m != k} e_m^2, with the linear weights d_k = 0.1, 0.6, 0.3
// folded into the candidate coefficients of the numerator.
template <typename T>
__device__ __forceinline__ T weno5u(T v1, T v2, T v3, T v4, T v5, T eps2)
{
    const T s1 = v2 - v1, s2 = v3 - v2, s3 = v4 - v3, s4 = v5 - v4;
    const T a1 = s2 - s1, a2 = s3 - s2, a3 = s4 - s3;
    const T b1 = (T)3 * s2 - s1, b2 = s2 + s3, b3 = s4 - (T)3 * s3;
    const T c = (T)(13.0 / 3.0), e4 = (T)4 * eps2;
    T e1 = b1 * b1 + (c * a1 * a1 + e4);
    T e2 = b2 * b2 + (c * a2 * a2 + e4);
    T e3 = b3 * b3 + (c * a3 * a3 + e4);
    if constexpr (sizeof(T) == 4) {
        // FP32: eps h^2 squared twice in the common denominator underflows on fine grids; any
        // common scale serves, so normalise by (about) the largest indicator: the difference of the
        // bit patterns negates its exponent (1/m to 12 %, for any normal m up to 2^125), at a
        // quarter of the hardware reciprocal's issue time
        const float m = fmaxf(fmaxf(e1, e2), e3);
        const T im = __builtin_bit_cast(float, 0x7ef00000u - __builtin_bit_cast(unsigned, m));
        e1 *= im; e2 *= im; e3 *= im;
    }
    e1 *= e1; e2 *= e2; e3 *= e3;
    const T p1 = e2 * e3, p2 = e1 * e3, p3 = e1 * e2;
    // 5 d_k q_k for d_k = 0.1, 0.6, 0.3, and 5 d_k below (a factor that leaves s3 and s4 alone)
    const T r1 = (T)(5.0 / 12.0) * s2 - (T)(1.0 / 6.0) * s1;
    const T r2 = (T)0.5 * s2 + s3;
    const T r3 = (T)-0.25 * s4 + s3;
    const T num = p1 * r1 + p2 * r2 + p3 * r3;
    const T den = (T)0.5 * p1 + (T)3 * p2 + (T)1.5 * p3;
    // FP32: the hardware reciprocal (about one ulp) is already at the precision of the FP32 sum;
    // FP64 refines it to full precision
    const T iw = sizeof(T) == 4 ? (T)__builtin_amdgcn_rcpf((float)den) : fast_rcp(den);
    return v3 + num * iw;
}

// regularised Heaviside of the two-phase mixture (Sec. 3.2.1): 0 below -e, 1 above e, smooth
// between
__device__ __forceinline__ double heaviside(double phi, double e)
{
    if (phi < -e) return 0.0;
    if (phi > e) return 1.0;
    return 0.5 * (1.0 + phi / e + sin(M_PI * phi / e) / M_PI);
}

}  // namespace evp
