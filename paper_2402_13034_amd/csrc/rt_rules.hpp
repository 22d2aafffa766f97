// Which way a call takes, where the sizes alone decide: plain functions of
// them, shared by the library and a host-side test that holds them against the
// measured times of both ways.
#pragma once
#include <math.h>
#include <stdint.h>

#ifndef RT_HD
#if defined(__HIPCC__)
#define RT_HD __host__ __device__
#else
#define RT_HD
#endif
#endif

namespace rt {

// A binned surface-area split above the surfaces' subtrees: in one workgroup, so
// up to RT_TOP_MAX surfaces.
constexpr int RT_TOP_MAX = 8192;
constexpr int RT_TOP_RES = 2048;   // surfaces whose boxes fit its LDS
RT_HD inline bool top_wanted(int64_t n_surf) { return n_surf >= 2 && n_surf <= RT_TOP_MAX; }

// The split of every surface, or of groups of 64 along a Morton order?  The
// first gives the better tree (us, traces of 10^6 rays at order 2: 1992 against
// 2414 for 8000 surfaces of 8 triangles; 929 and 961 for 1000 of 2) and costs a
// build 70 us at 100 surfaces, 180 at 600, 300 to 370 at 2000, whose boxes fit
// its LDS, and 430 at 3000, 670 at 5000, 990 at 8000; the groups 80 at 600, 110 at
// 2000, 220 at 8000.  Every surface is split where a build and one small trace
// take no longer than they did with one linear BVH for the whole scene and its
// atomic refit (us before / full / grouped: 300 surfaces of 8 triangles 841 /
// 649 / 621, 8000 of 8 1975 / 1753 / 1055; to within 2 % up to 256 surfaces: 192
// of 1 571 / 583 / 573), so not for surfaces of few triangles by the hundred
// (592 of 1 616 / 631 / 560, 996 of 2 687 / 706 / 599) or thousand (3000 of 2 970 /
// 1063 / 810, 8000 of 2 1235 / 1646 / 940).
RT_HD inline bool top_full(int64_t n_surf, int64_t n_tri) { return n_surf <= 256 || n_tri >= 8 * n_surf; }

// Discovery with four lanes per ray (k_discover_quad) instead of a wave walking
// for 64 rays (k_discover)?  The wave visits the union of its rays' nodes, one
// after the other: with few rays against the triangles that is many times a
// ray's own nodes, and the launch has too few waves to hide the chain.  Its time
// falls with the rays' density and grows with the order, as the first bounce
// alone is coherent; four lanes a ray take 1.55 us per 1000 rays at any order.
// The rays from which the wave is faster go with n_tri^0.4, by order (both
// sources' kernels, us, wave / four lanes):
//   order 1  1908 triangles 5 10^4 rays 93 / 100, 17 000 14 10^4 226 / 235,
//            49 000 14 10^4 357 / 238, 2 10^5 258 / 320
//   order 2  1908 7 10^4 189 / 139, 14 10^4 150 / 245; 17 000 14 10^4 519 / 252, 3 10^5 366 / 490
//   order 3  1908 10^5 284 / 192, 2 10^5 267 / 339; 17 000 3 10^5 595 / 499, 4 10^5 528 / 645
//   order 5  1908 2 10^5 1402 / 1090, 4 10^5 1292 / 1378
// and from 5 10^5 on (10^6 rays and 1.08 million triangles 2614 / 4086).  What one line gives
// up: an office floor's rays are coherent (103 000 triangles, order 2, 3 10^5
// rays 364 / 493), clutter's are not (200 000, order 3, 6 10^5 2125 / 1017).
inline bool sparse_rays(int64_t n_rays, int64_t n_tri, int order)
{
    const double by_order[4] = {2100.0, 4000.0, 6500.0, 12000.0};
    const double most = by_order[order < 1 ? 0 : order > 4 ? 3 : order - 1] * pow((double)n_tri, 0.4);
    return n_tri >= 64 && n_rays <= 500000 && (double)n_rays <= most;
}

// The matrix-core sum on tiles of 64 receivers x 64 configurations (k_sum_few)
// instead of 256 rows (128 receivers) x 256?  kend: the contraction, M for real
// Gamma, 2 M for complex.  A large tile is eight small ones and takes its CU 2.5
// times as long as a small one (45 against 18 ns a k), and Gamma's own split
// costs 8 us more.  While the large tiles leave CUs idle, four small tiles a CU
// for every large one are still the faster way up to 512 k (4096 receivers x 127
// complex: 29 against 37 us at 1024 configurations, 49 against 41 at 2048), two
// above (1024 complex elements, 16384 receivers: 75 against 113 us at 100
// configurations, 162 against 113 at 256).  Where the large ones fill the chip
// each column of small tiles reads H's split again, so four are only faster up
// to 256 k and 2^24 receivers x k (100 configurations, small / large: 32768
// receivers x 127 complex 39 / 46 us, x 200 complex 55 / 51; 65536 x 127 complex 66 / 68,
// x 331 real 89 / 78, x 256 complex 118 / 96).  Half as many for three products,
// whose stages leave room for one workgroup a CU.
inline bool small_tiles(int64_t R, int64_t C, int64_t kend, bool three, int64_t cus)
{
    const int64_t large = (2 * R + 255) / 256 * ((C + 255) / 256);
    const int64_t small = (R + 63) / 64 * ((C + 63) / 64);
    const bool filled = large >= cus && !three;
    const bool four = kend <= 512 && (!filled || (kend <= 256 && R * kend < ((int64_t)1 << 24)));
    const int64_t per = (four ? 4 : 2) / (three ? 2 : 1);
    return small <= per * cus * ((large + cus - 1) / cus) && small < ((int64_t)1 << 31);
}

}  // namespace rt
