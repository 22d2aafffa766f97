// Host check of the kernels' FP64 division and square root at the ends of the
// range they state: exact while the numbers and the residuals they correct by
// stay normal, and what lies beyond gives no path a wrong decision.
#include <initializer_list>
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
// random mantissa but all ones, exponent in [lo, hi]
static double value(int lo, int hi)
{
    uint64_t m = rnd() & ((1ull << 52) - 2);
    const uint64_t b = (uint64_t)(1023 + lo + (int)(rnd() % (uint64_t)(hi - lo + 1))) << 52 | m;
    double d;
    memcpy(&d, &b, 8);
    return d;
}

int main()
{
    long bad = 0;
    double L, il;
    for (long i = 0; i < 2000000; ++i) {
        // squared distances of 10^-144 to 10^154 m
        const double x = value(-960, 1022);
        rt::sqrt_refine(x, 1.0 / sqrt(x) * (1.0 + ldexp((double)(rnd() >> 12), -75)), &L, &il);
        if (L != sqrt(x) || fabs(il - 1.0 / L) > ldexp(1.0 / L, -52)) ++bad;
        // a plane's numerator and denominator: products of coordinates up to 10^120
        const double a = value(-700, 400), b = value(-300, 400);
        if (rt::div_refine(a, b, 1.0 / b * (1.0 + ldexp((double)(rnd() >> 12), -75))) != a / b) ++bad;
    }
    // the estimate of 1 / sqrt(x) is that of 1e-300 below it: shorter than any leg that is searched
    for (double x : {0.0, 4.9e-324, 1e-310, 1e-301}) {
        rt::sqrt_refine(x, 1e150, &L, &il);
        if (!(L >= 0.0 && L < 1e-149) || !isfinite(il)) ++bad;
    }
    // an infinite square has no finite root: not a number, which no comparison accepts
    rt::sqrt_refine(INFINITY, 0.0, &L, &il);
    if (!isnan(L) || L - 1e-4 > 1e-4) ++bad;
    if (!isnan(rt::div_refine(1.0, 0.0, INFINITY))) ++bad;
    printf("%ld wrong\n", bad);
    return bad ? 1 : 0;
}
