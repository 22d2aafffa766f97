// Host check of the rules by size: at measured points (us) each takes the way
// that its comment says it takes.
#include <stdio.h>

#include "../../paper_2402_13034_amd/csrc/rt_rules.hpp"

static int bad = 0;
static void expect(const char* rule, bool got, bool want, long a, long b, long c = 0)
{
    if (got == want) return;
    printf("%s(%ld, %ld, %ld) is %d\n", rule, a, b, c, (int)got);
    ++bad;
}

// surfaces, triangles; a build and one small trace: one linear BVH with the atomic refit, every surface split, groups
static const long top[][5] = {
    {192, 192, 571, 583, 573},        {96, 192, 545, 531, 517},         {96, 768, 657, 561, 566},
    {592, 592, 616, 631, 560},        {1192, 1192, 659, 707, 582},      {1992, 1992, 700, 788, 620},
    {3992, 3992, 881, 1117, 714},     {5992, 5992, 963, 1385, 857},     {596, 1192, 661, 670, 582},
    {996, 1992, 687, 706, 599},       {1996, 3992, 876, 889, 680},      {2996, 5992, 970, 1063, 810},
    {4996, 9992, 1076, 1307, 870},    {7996, 15992, 1235, 1646, 940},   {296, 2368, 841, 649, 621},
    {596, 4768, 1013, 872, 771},      {996, 7968, 1084, 918, 811},      {1996, 15968, 1317, 1070, 869},
    {2996, 23968, 1484, 1135, 880},   {4996, 39968, 1664, 1387, 953},   {7996, 63968, 1975, 1753, 1055},
    {7996, 255872, 4393, 2007, 1318},
};

int main()
{
    // every surface where that is faster than before there was a split, groups where it is slower (2 % either way is left
    // out), and what is taken is never slower
    for (const auto& p : top) {
        const bool full = rt::top_full(p[0], p[1]);
        if (100 * p[3] < 98 * p[2]) expect("top_full", full, true, p[0], p[1]);
        if (1000 * p[3] > 1025 * p[2]) expect("top_full", full, false, p[0], p[1]);
        if (1000 * (full ? p[3] : p[4]) > 1025 * p[2]) expect("top_full slower", full, !full, p[0], p[1]);
    }
    expect("top_wanted", rt::top_wanted(1), false, 1, 0);
    expect("top_wanted", rt::top_wanted(2), true, 2, 0);
    expect("top_wanted", rt::top_wanted(8192), true, 8192, 0);
    expect("top_wanted", rt::top_wanted(8193), false, 8193, 0);
    printf("%d wrong\n", bad);
    return bad ? 1 : 0;
}
