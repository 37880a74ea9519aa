// quotient.hpp -- division by the call's temperature.  Plain C++ for the host
// and the device compiler alike, so that the host can check it against its own
// division.
#pragma once

#if defined(__HIP__)
#define ROI_HD __host__ __device__ __forceinline__
#else
#define ROI_HD inline
#endif

namespace roi {

// a / b correctly rounded, given y = RN(1 / b): q = RN(a y) is within 1.5 ulp
// of a / b; one correction by the residual a - q b leaves it within one ulp,
// where the next residual is exact and the correction by it rounds correctly
// (Markstein, IBM J. Res. Dev. 34, 1990: with y the rounded reciprocal, q
// within an ulp and the residual exact, RN(q + r y) = RN(a / b)).  It needs
// every residual above underflow and no overflow: kQuotientLo <= |b| <=
// kQuotientHi and 2^-100 <= |a| <= kQuotientMax; a = 0 gives a zero.  For a
// smaller nonzero |a| the residual may lose bits and the last bit of a
// quotient below 2^-80 with them.
constexpr float kQuotientLo = 0x1p-20f, kQuotientHi = 0x1p20f, kQuotientMax = 0x1p100f;

ROI_HD float quotient(float a, float b, float y)
{
    float q = a * y;
    q = __builtin_fmaf(__builtin_fmaf(-q, b, a), y, q);
    return __builtin_fmaf(__builtin_fmaf(-q, b, a), y, q);
}

} // namespace roi
