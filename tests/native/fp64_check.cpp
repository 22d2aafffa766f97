// Host check of the kernels' FP64 division, square root and reciprocal: from
// estimates off by up to 2^-22 they give the correctly rounded results, except
// for divisors with all fraction bits set, where one unit is allowed.
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "../../paper_2402_13034_amd/csrc/rt_fp64_core.hpp"

static uint64_t state = 88172645463325252ull;
static uint64_t rnd()
{
    state ^= state << 13;
    state ^= state >> 7;
    state ^= state << 17;
    return state;
}
// random sign and mantissa (now and then all ones or all zeros), exponent in [lo, hi]
static double value(int lo, int hi)
{
    uint64_t m = rnd() & ((1ull << 52) - 1);
    const uint64_t pick = rnd() % 64;
    if (pick == 0) m = (1ull << 52) - 1;
    if (pick == 1) m = 0;
    const uint64_t b = (uint64_t)(1023 + lo + (int)(rnd() % (uint64_t)(hi - lo + 1))) << 52 | m;
    double d;
    memcpy(&d, &b, 8);
    return rnd() & 1 ? -d : d;
}
static bool all_ones(double x)
{
    uint64_t b;
    memcpy(&b, &x, 8);
    return (b & ((1ull << 52) - 1)) == (1ull << 52) - 1;
}
// got is want, or within one unit of it where the divisor is the exception
static bool right(double got, double want, double divisor)
{
    if (got == want) return true;
    return all_ones(divisor) && (got == nextafter(want, INFINITY) || got == nextafter(want, -INFINITY));
}
static double off() { return 1.0 + ldexp((double)(rnd() >> 11) / 4503599627370496.0 - 1.0, -22); }

int main()
{
    long bad = 0;
    for (long i = 0; i < 4000000; ++i) {
        const bool wide = i % 2;
        const double a = value(wide ? -200 : -30, wide ? 60 : 30), b = value(wide ? -200 : -20, wide ? 60 : 20);
        if (rt::div_by(a, b, 1.0 / b) != a / b) ++bad;
        if (!right(rt::div_refine(a, b, 1.0 / b * off()), a / b, b)) ++bad;
        const double x = fabs(value(wide ? -400 : -30, wide ? 60 : 30));
        double L, il;
        rt::sqrt_refine(x, 1.0 / sqrt(x) * off(), &L, &il);
        if (L != sqrt(x) || !right(il, 1.0 / L, L)) ++bad;
    }
    double L, il;
    rt::sqrt_refine(0.0, 1e150, &L, &il);
    if (L != 0.0 || !(il > 0.0) || isinf(il)) ++bad;
    printf("%ld wrong\n", bad);
    return bad ? 1 : 0;
}
