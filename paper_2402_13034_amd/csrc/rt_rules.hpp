// Which way a call takes, where the sizes alone decide: plain functions of
// them, shared by the library and a host-side test that holds them against the
// measured times of both ways.
#pragma once
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

}  // namespace rt
