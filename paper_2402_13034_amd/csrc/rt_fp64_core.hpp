// FP64 division, square root and reciprocal without the range scaling of the
// general operations: an estimate, refined until the last correction rounds
// correctly (Markstein, "Computation of elementary functions on the IBM RISC
// System/6000 processor", IBM J. R&D 34, 1990), so the results are those of
// a / b, sqrt(x) and 1.0 / sqrt(x) wherever the numbers and the residuals stay
// normal.  Scene vertices are FP32 of at most 1e6 m (products of their
// differences stay above 1e-91); the points a caller gives (antennas, receivers,
// elements) are not bounded: legs from 1e-144 to 1.3e154 m are exact.  A shorter
// one comes out shorter than any that is searched, a longer one as NaN where a
// root would be infinite: blocked by nothing either way, and only the length of
// such a kept path shows it.  A divisor with all 52 fraction bits set is the
// method's one exception: its reciprocal may come out one unit below.
// Shared by the kernels (estimates from v_rcp_f64 and v_rsq_f64) and their
// host-side tests.
#pragma once

#ifndef RT_HD
#if defined(__HIPCC__)
#define RT_HD __host__ __device__
#else
#define RT_HD
#endif
#endif

namespace rt {

// a / b, y = 1 / b correctly rounded
RT_HD inline double div_by(double a, double b, double y)
{
    const double q = a * y;
    return __builtin_fma(__builtin_fma(-b, q, a), y, q);
}

// a / b from an estimate y of 1 / b (22 bits or more)
RT_HD inline double div_refine(double a, double b, double y)
{
    y = __builtin_fma(y, __builtin_fma(-b, y, 1.0), y);
    y = __builtin_fma(y, __builtin_fma(-b, y, 1.0), y);
    return div_by(a, b, y);
}

// L = sqrt(x) and il = 1 / L from an estimate y of 1 / sqrt(x); x = 0 with any
// finite y gives L = 0 and a finite il
RT_HD inline void sqrt_refine(double x, double y, double* L, double* il)
{
    double g = x * y, h = 0.5 * y;
    const double r = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, r, g);
    h = __builtin_fma(h, r, h);
    g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
    g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
    *L = g;
    double z = h + h;
    z = __builtin_fma(z, __builtin_fma(-g, z, 1.0), z);
    *il = __builtin_fma(__builtin_fma(-g, z, 1.0), z, z);
}

}  // namespace rt
