// Scene upload and linear BVH build on the device.
//
// LBVH after Karras, "Maximizing Parallelism in the Construction of BVHs,
// Octrees, and k-d Trees" (HPG 2012): 30-bit Morton codes of triangle
// centroids with the triangle index appended (unique 62-bit keys), radix
// sort, one thread per internal node finds its key range and split, then the
// node boxes: bottom-up within tiles of leaves, by leaf range above them.
// Node boxes are inflated so that the FP32 slab test is conservative with
// respect to the exact ray/triangle formula.
//
// Layouts (leaf slot = rank of the triangle's key):
//   tri4  [3 * n]: (v0.xyz, id), (e1.xyz, surface), (e2.xyz, 0)
//   nodes [4 * (n - 1)]: (loL.xyz, childL), (hiL.xyz, childR), (loR.xyz, -), (hiR.xyz, -)
//   child >= 0: internal node; child < 0: leaf slot ~child.
// Surfaces: s_tris groups triangle indices by surface (ascending), s_ptr the
// CSR offsets, s_plane the plane of each surface's lowest-numbered triangle.
#pragma clang fp contract(off)

#include <algorithm>
#include <cstring>
#include <vector>

#include "rt_host.hpp"
#include "rt_lbvh_core.hpp"

namespace rt {

__device__ __forceinline__ unsigned f2ord(float f)
{
    unsigned u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float ord2f(unsigned u)
{
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

// bounds[0..2] min centroid, [3..5] max centroid, [6..8] min vertex, [9..11] max vertex
__device__ __forceinline__ unsigned wave_umin(unsigned v)
{
    for (int o = 32; o > 0; o >>= 1) v = min(v, (unsigned)__shfl_xor((int)v, o, 64));
    return v;
}
__device__ __forceinline__ unsigned wave_umax(unsigned v)
{
    for (int o = 32; o > 0; o >>= 1) v = max(v, (unsigned)__shfl_xor((int)v, o, 64));
    return v;
}

// FP64 vertices and their 2-D projection, reflection coefficients, surface
// ids and sort keys (surface above triangle), centroids; bounds of the
// centroids and of the vertices (order-preserving unsigned keys) and the
// largest surface id.  Every block ends in 13 atomics on the same few words,
// which serialise across the XCDs: at most PREP_BLOCKS blocks stride over the
// triangles and reduce in LDS first (200 000 triangles: 444 us with 12 atomics
// per wave, 30 us so).
constexpr int PREP_B = 256, PREP_BLOCKS = 512;
__global__ __launch_bounds__(PREP_B) void k_scene_prep(const float* V, const int32_t* T, const int32_t* surf_in,
                                                       const float* rr, const float* ri, int64_t nv, int64_t nt,
                                                       double* v64, float2* refl, int32_t* surf, float4* cent,
                                                       uint64_t* skeys, unsigned* bounds, int32_t* bad,
                                                       int32_t* n_surf, double* proj, int32_t* axes)
{
    __shared__ unsigned red[PREP_B / 64][13];
    unsigned mn[6], mx[6];   // minima and maxima of the centroids (0..2) and the vertices (3..5)
    for (int k = 0; k < 6; ++k) {
        mn[k] = 0xffffffffu;
        mx[k] = 0u;
    }
    unsigned smax = 0u, flags = 0u;
    for (int64_t t = (int64_t)blockIdx.x * PREP_B + threadIdx.x; t < nt; t += (int64_t)gridDim.x * PREP_B) {
        float c[3] = {0, 0, 0};
        double w[9];
        for (int j = 0; j < 3; ++j) {
            int32_t vi = T[3 * t + j];
            if (vi < 0 || vi >= nv) {
                flags |= 1u;
                vi = 0;
            }
            for (int k = 0; k < 3; ++k) {
                const float x = V[3 * (int64_t)vi + k];
                if (!(x == x) || fabsf(x) > 1e6f) flags |= 2u;
                w[3 * j + k] = (double)x;
                v64[9 * t + 3 * j + k] = (double)x;
                c[k] += x;
                const unsigned u = f2ord(x);
                mn[3 + k] = min(mn[3 + k], u);
                mx[3 + k] = max(mx[3 + k], u);
            }
        }
        triangle_projection(w, proj + 6 * t, axes + t);
        refl[t] = make_float2(rr[t], ri[t]);
        const int32_t sf = surf_in[t];
        surf[t] = sf;
        // surface ids are clamped to 0..nt-1 (larger ones are reported as invalid)
        if (sf < 0 || sf >= nt) flags |= 4u;
        const int32_t sc = sf < 0 ? 0 : (sf >= nt ? (int32_t)(nt - 1) : sf);
        skeys[t] = ((uint64_t)(uint32_t)sc << 32) | (uint64_t)t;
        smax = max(smax, (unsigned)sc + 1u);
        for (int k = 0; k < 3; ++k) {
            c[k] = c[k] / 3.0f;
            const unsigned u = f2ord(c[k]);
            mn[k] = min(mn[k], u);
            mx[k] = max(mx[k], u);
        }
        cent[t] = make_float4(c[0], c[1], c[2], 0.0f);
    }
    if (flags) atomicOr(bad, (int32_t)flags);
    const int wave = threadIdx.x >> 6;
    for (int k = 0; k < 6; ++k) {
        const unsigned a = wave_umin(mn[k]), b = wave_umax(mx[k]);
        if ((threadIdx.x & 63) == 0) {
            red[wave][k] = a;
            red[wave][6 + k] = b;
        }
    }
    const unsigned sm = wave_umax(smax);
    if ((threadIdx.x & 63) == 0) red[wave][12] = sm;
    __syncthreads();
    if (threadIdx.x < 13) {
        const int k = threadIdx.x;
        unsigned v = red[0][k];
        for (int q = 1; q < PREP_B / 64; ++q) v = k < 6 ? min(v, red[q][k]) : max(v, red[q][k]);
        // bounds: centroid minima, maxima, vertex minima, maxima (three words each)
        if (k < 6)
            atomicMin(&bounds[k < 3 ? k : k + 3], v);
        else if (k < 12)
            atomicMax(&bounds[k < 9 ? k - 3 : k], v);
        else
            atomicMax(n_surf, (int32_t)v);
    }
}

// spread the low 21 bits of v to every third bit of 63 (bit i -> bit 3 i)
__device__ __forceinline__ uint64_t expand21(uint64_t v)
{
    v &= 0x1fffffull;
    v = (v | v << 32) & 0x1f00000000ffffull;
    v = (v | v << 16) & 0x1f0000ff0000ffull;
    v = (v | v << 8) & 0x100f00f00f00f00full;
    v = (v | v << 4) & 0x10c30c30c30c30c3ull;
    v = (v | v << 2) & 0x1249249249249249ull;
    return v;
}

// Two-word sort keys: word 0 the triangle index, word 1 the 63-bit Morton code
// of the centroid (21 bits per axis over the scene bounds); sorted on word 1,
// stably, so equal codes stay in index order (the tie-break of the unique keys).
// Block 0 also writes the vertices' bounds as floats (lower x y z, upper x y z).
__global__ void k_morton(const float4* cent, const unsigned* bounds, int64_t nt, uint64_t* keys, float* box)
{
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < 6) box[t] = ord2f(bounds[6 + t]);
    if (t >= nt) return;
    float lo[3], ext[3];
    for (int k = 0; k < 3; ++k) {
        lo[k] = ord2f(bounds[k]);
        float hi = ord2f(bounds[3 + k]);
        ext[k] = hi - lo[k];
    }
    float4 c = cent[t];
    float cc[3] = {c.x, c.y, c.z};
    uint64_t q[3];
    for (int k = 0; k < 3; ++k) {
        float u = ext[k] > 0.0f ? (cc[k] - lo[k]) / ext[k] : 0.5f;
        u = fminf(fmaxf(u, 0.0f), 1.0f);
        q[k] = (uint64_t)fminf(u * 2097152.0f, 2097151.0f);
    }
    keys[2 * t] = (uint64_t)t;
    keys[2 * t + 1] = (expand21(q[0]) << 2) | (expand21(q[1]) << 1) | expand21(q[2]);
}

struct Box6 {
    float lo[3], hi[3];
};

__device__ __forceinline__ int64_t clamp_index(int32_t v, int64_t n) { return v < 0 ? 0 : (v >= n ? n - 1 : v); }

// Leaf data in sorted order.  Box padding: 1e-5 of the scene extent + 1e-6 m
// + 1e-5 |x| (indices are clamped: malformed input is reported after the build).
__global__ void k_leaves(const uint64_t* keys, const float* V, const int32_t* T, const int32_t* surf, int64_t nv,
                         int64_t nt, const unsigned* bounds, float4* tri4, float* lbox)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nt) return;
    float ext = 0.0f;
    for (int k = 0; k < 3; ++k) ext = fmaxf(ext, ord2f(bounds[9 + k]) - ord2f(bounds[6 + k]));
    const float pad = 1e-5f * ext + 1e-6f;
    int32_t t = (int32_t)keys[2 * i];   // word 0 of the sorted key: the triangle index
    const float* a = V + 3 * clamp_index(T[3 * t + 0], nv);
    const float* b = V + 3 * clamp_index(T[3 * t + 1], nv);
    const float* c = V + 3 * clamp_index(T[3 * t + 2], nv);
    tri4[3 * i + 0] = make_float4(a[0], a[1], a[2], __int_as_float(t));
    tri4[3 * i + 1] = make_float4(b[0] - a[0], b[1] - a[1], b[2] - a[2], __int_as_float(surf[t]));
    tri4[3 * i + 2] = make_float4(c[0] - a[0], c[1] - a[1], c[2] - a[2], 0.0f);
    for (int k = 0; k < 3; ++k) {
        float lo = fminf(a[k], fminf(b[k], c[k]));
        float hi = fmaxf(a[k], fmaxf(b[k], c[k]));
        float p = pad + 1e-5f * fmaxf(fabsf(lo), fabsf(hi));
        lbox[6 * i + k] = lo - p;
        lbox[6 * i + 3 + k] = hi + p;
    }
}

// Leaves per tile of the refit (one workgroup each).
constexpr int RT_REFIT_TILE = 2048;
static_assert((RT_REFIT_TILE & (RT_REFIT_TILE - 1)) == 0, "tiles are found by division");

// One thread per internal node: children, parent links, the leaf range below
// the node; the nodes whose leaves span several refit tiles are listed (in no
// fixed order) for k_refit_cross.
__global__ void k_karras(const uint64_t* keys, int64_t n, int32_t* child, int32_t* parent_int,
                         int32_t* parent_leaf, int2* range, int32_t* cross, int32_t* n_cross)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n - 1) return;
    if (i == 0) parent_int[0] = -1;   // the root; every other node and every leaf gets its parent below
    int32_t cl, cr, first, last;
    lbvh_node<2>(keys, n, i, &cl, &cr, &first, &last);
    if (cl < 0) parent_leaf[~cl] = (int32_t)i;
    else parent_int[cl] = (int32_t)i;
    if (cr < 0) parent_leaf[~cr] = (int32_t)i;
    else parent_int[cr] = (int32_t)i;
    child[2 * i] = cl;
    child[2 * i + 1] = cr;
    range[i] = make_int2(first, last);
    if (first / RT_REFIT_TILE != last / RT_REFIT_TILE) cross[atomicAdd(n_cross, 1)] = (int32_t)i;
}

// Node boxes, part 1: one workgroup per tile of consecutive leaves computes
// the nodes whose leaves all lie in its tile, in the leaf-to-root order with
// every shared word in LDS (a node with that property has its index in the
// tile too).  A walker carries the box of the node it comes from in registers
// and leaves it in the parent's slot for that side; per node one word holds
// the parent link (plus one, low 29 bits) with the arrival count above it, so
// one LDS atomic per level both counts the arrival and yields the next node.
// The first arrival at a node stops; the second has both boxes and takes the
// union.  A node that does not see exactly two arrivals marks the tree
// inconsistent (flag 8).  The box of the whole tile goes to tbox.
// A tree in one tile is complete after this.  The walk over the whole device
// needs agent-scope fences at every level, each of which flushes an XCD's L2:
// 200 000 triangles took 1707 us that way; 22 us here and 29 us in part 2.
constexpr uint32_t RT_UP_LINK = (1u << 29) - 1;
constexpr uint32_t RT_UP_CROSS = 0xffffffffu;   // the node's leaves span several tiles
__global__ __launch_bounds__(1024) void k_refit_tiles(const int32_t* child, const int32_t* parent_int,
                                                      const int32_t* parent_leaf, const int2* range,
                                                      const float* lbox, float4* nodes, int64_t n, float* tbox,
                                                      int32_t* bad)
{
    __shared__ float side[RT_REFIT_TILE * 12];   // [node][left, right][lo xyz, hi xyz]
    __shared__ int32_t ch[2 * RT_REFIT_TILE];
    __shared__ uint32_t up[RT_REFIT_TILE];
    __shared__ float wbox[16][6];
    const int t0 = (int)blockIdx.x * RT_REFIT_TILE;
    const int nl = (int)min((int64_t)RT_REFIT_TILE, n - t0);           // leaves of the tile
    const int ni = (int)min((int64_t)RT_REFIT_TILE, n - 1 - t0);       // node indices of the tile
    for (int q = threadIdx.x; q < ni; q += blockDim.x) {
        const int p = t0 + q;
        const int2 r = range[p];
        const int32_t par = parent_int[p];
        ch[2 * q] = child[2 * p];
        ch[2 * q + 1] = child[2 * p + 1];
        up[q] = r.x < t0 || r.y >= t0 + nl ? RT_UP_CROSS
                                           : (par >= -1 && par < n - 1 ? (uint32_t)(par + 1) : RT_UP_LINK);
    }
    __syncthreads();
    float tb[6] = {3e38f, 3e38f, 3e38f, -3e38f, -3e38f, -3e38f};
    for (int i = threadIdx.x; i < nl; i += blockDim.x) {
        float b[6];
        for (int k = 0; k < 6; ++k) b[k] = lbox[6 * (int64_t)(t0 + i) + k];
        for (int k = 0; k < 3; ++k) {
            tb[k] = fminf(tb[k], b[k]);
            tb[3 + k] = fmaxf(tb[3 + k], b[3 + k]);
        }
        int32_t from = ~(t0 + i);
        int32_t p = parent_leaf[t0 + i];
        while (p >= t0 && p - t0 < ni) {
            const int q = p - t0;
            if (up[q] == RT_UP_CROSS) break;
            const int32_t cl = ch[2 * q], cr = ch[2 * q + 1];
            const int me = from == cl ? 0 : 1;
            if (me == 1 && from != cr) {
                atomicOr(bad, 8);
                break;
            }
            float* mine = side + 12 * q + 6 * me;
            for (int k = 0; k < 6; ++k) mine[k] = b[k];
            const uint32_t old =
                __hip_atomic_fetch_add(&up[q], 1u << 29, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
            if ((old >> 29) == 0) break;   // first arrival: the other child completes p
            const float* l = side + 12 * q;
            const float* r = l + 6;
            nodes[4 * (int64_t)p + 0] = make_float4(l[0], l[1], l[2], __int_as_float(cl));
            nodes[4 * (int64_t)p + 1] = make_float4(l[3], l[4], l[5], __int_as_float(cr));
            nodes[4 * (int64_t)p + 2] = make_float4(r[0], r[1], r[2], 0.0f);
            nodes[4 * (int64_t)p + 3] = make_float4(r[3], r[4], r[5], 0.0f);
            for (int k = 0; k < 3; ++k) {
                b[k] = fminf(l[k], r[k]);
                b[3 + k] = fmaxf(l[3 + k], r[3 + k]);
            }
            from = p;
            p = (int32_t)(old & RT_UP_LINK) - 1;
        }
    }
    for (int o = 32; o > 0; o >>= 1)
        for (int k = 0; k < 6; ++k) {
            const float v = __shfl_xor(tb[k], o, 64);
            tb[k] = k < 3 ? fminf(tb[k], v) : fmaxf(tb[k], v);
        }
    if ((threadIdx.x & 63) == 0)
        for (int k = 0; k < 6; ++k) wbox[threadIdx.x >> 6][k] = tb[k];
    __syncthreads();
    for (int q = threadIdx.x; q < ni; q += blockDim.x)
        if (up[q] != RT_UP_CROSS && (up[q] >> 29) != 2) atomicOr(bad, 8);
    if (threadIdx.x < 6) {
        const int k = threadIdx.x;
        float v = wbox[0][k];
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) v = k < 3 ? fminf(v, wbox[w][k]) : fmaxf(v, wbox[w][k]);
        tbox[6 * (int64_t)blockIdx.x + k] = v;
    }
}

// Union over the leaves first..last of a wave's lanes: the leaves of the two
// end tiles one by one, the tiles between by their boxes (the same minima and
// maxima whatever the order).
__device__ __forceinline__ void range_box(const float* lbox, const float* tbox, int first, int last, float* b)
{
    const int lane = threadIdx.x & 63;
    for (int k = 0; k < 3; ++k) {
        b[k] = 3e38f;
        b[3 + k] = -3e38f;
    }
    auto take = [&](const float* src) {
        for (int k = 0; k < 3; ++k) {
            b[k] = fminf(b[k], src[k]);
            b[3 + k] = fmaxf(b[3 + k], src[3 + k]);
        }
    };
    const int ta = first / RT_REFIT_TILE, tz = last / RT_REFIT_TILE;
    const int ea = ta == tz ? last : (ta + 1) * RT_REFIT_TILE - 1;
    for (int i = first + lane; i <= ea; i += 64) take(lbox + 6 * (int64_t)i);
    for (int t = ta + 1 + lane; t < tz; t += 64) take(tbox + 6 * (int64_t)t);
    if (ta != tz)
        for (int i = tz * RT_REFIT_TILE + lane; i <= last; i += 64) take(lbox + 6 * (int64_t)i);
    for (int o = 32; o > 0; o >>= 1)
        for (int k = 0; k < 6; ++k) {
            const float v = __shfl_xor(b[k], o, 64);
            b[k] = k < 3 ? fminf(b[k], v) : fmaxf(b[k], v);
        }
}

// Node boxes, part 2: the nodes whose leaves span several tiles, one wave
// each, every child's box straight from its leaf range (no order between
// nodes, so no fences).
__global__ __launch_bounds__(256) void k_refit_cross(const int32_t* cross, const int32_t* n_cross,
                                                     const int32_t* child, const int32_t* parent_int,
                                                     const int32_t* parent_leaf, const int2* range,
                                                     const float* lbox, const float* tbox, float4* nodes,
                                                     int32_t* bad)
{
    const int lane = threadIdx.x & 63;
    const int nc = *n_cross;
    for (int e = (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)); e < nc;
         e += (int)(gridDim.x * (blockDim.x >> 6))) {
        const int p = cross[e];
        const int2 r = range[p];
        const int32_t cl = child[2 * p], cr = child[2 * p + 1];
        const int g = cl < 0 ? ~cl : cl;   // last leaf of the left child
        float l[6], h[6];
        range_box(lbox, tbox, r.x, g, l);
        range_box(lbox, tbox, g + 1, r.y, h);
        if (lane == 0) {
            nodes[4 * (int64_t)p + 0] = make_float4(l[0], l[1], l[2], __int_as_float(cl));
            nodes[4 * (int64_t)p + 1] = make_float4(l[3], l[4], l[5], __int_as_float(cr));
            nodes[4 * (int64_t)p + 2] = make_float4(h[0], h[1], h[2], 0.0f);
            nodes[4 * (int64_t)p + 3] = make_float4(h[3], h[4], h[5], 0.0f);
            const int32_t pl = cl < 0 ? parent_leaf[~cl] : parent_int[cl];
            const int32_t pr = cr < 0 ? parent_leaf[~cr] : parent_int[cr];
            if (pl != p || pr != p) atomicOr(bad, 8);
        }
    }
}

// 4-wide nodes: every internal node of even depth lists its grandchildren
// (a leaf child stands for itself).  Boxes are copied from the binary nodes.
// Also the tree depth: the deepest leaf lies one below the deepest internal
// node (a broken parent chain gives 2^20).
__global__ void k_node4(const int32_t* child, const int32_t* parent_int, const float4* nodes, const float4* tri4,
                        int64_t ni, float4* node4, int32_t* maxd)
{
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = n < ni;
    int d = 0;
    int32_t p = live ? parent_int[n] : -1;
    for (; p >= 0 && p < ni && d < 4096; p = parent_int[p]) ++d;
    const unsigned dl = !live ? 0u : (p != -1 ? (1u << 20) : (unsigned)d + 1u);
    const unsigned dm = wave_umax(dl);
    if ((threadIdx.x & 63) == 0 && dm > 0) atomicMax(maxd, (int32_t)dm);
    if (!live || (d & 1)) return;
    float lo[4][3], hi[4][3];
    int32_t ref[4];
    int cnt = 0;
    for (int side = 0; side < 2; ++side) {
        const int32_t c = child[2 * n + side];
        const float4 l = nodes[4 * n + 2 * side], h = nodes[4 * n + 2 * side + 1];
        if (c < 0) {
            lo[cnt][0] = l.x; lo[cnt][1] = l.y; lo[cnt][2] = l.z;
            hi[cnt][0] = h.x; hi[cnt][1] = h.y; hi[cnt][2] = h.z;
            ref[cnt++] = c;
        } else {
            for (int g = 0; g < 2; ++g) {
                const float4 gl = nodes[4 * c + 2 * g], gh = nodes[4 * c + 2 * g + 1];
                lo[cnt][0] = gl.x; lo[cnt][1] = gl.y; lo[cnt][2] = gl.z;
                hi[cnt][0] = gh.x; hi[cnt][1] = gh.y; hi[cnt][2] = gh.z;
                ref[cnt++] = child[2 * c + g];
            }
        }
    }
    for (int j = cnt; j < 4; ++j) {
        lo[j][0] = lo[j][1] = lo[j][2] = 0.0f;   // masked out by the reference
        hi[j][0] = hi[j][1] = hi[j][2] = 0.0f;
        ref[j] = 0x7fffffff;
    }
    float4* q = node4 + 8 * n;
    for (int a = 0; a < 3; ++a) {
        q[2 * a] = make_float4(lo[0][a], lo[1][a], lo[2][a], lo[3][a]);
        q[2 * a + 1] = make_float4(hi[0][a], hi[1][a], hi[2][a], hi[3][a]);
    }
    q[6] = make_float4(__int_as_float(ref[0]), __int_as_float(ref[1]), __int_as_float(ref[2]),
                       __int_as_float(ref[3]));
    // surface of each leaf entry (-1 for inner and unused entries): walks that ignore a surface
    // drop its leaves without visiting them
    int lsf[4];
    for (int j = 0; j < 4; ++j)
        lsf[j] = (ref[j] < 0 && ref[j] != 0x7fffffff) ? __float_as_int(tri4[3 * (int64_t)(~ref[j]) + 1].w) : -1;
    q[7] = make_float4(__int_as_float(lsf[0]), __int_as_float(lsf[1]), __int_as_float(lsf[2]), __int_as_float(lsf[3]));
}

// CSR over surfaces from the sorted (surface, triangle) keys; an unused id
// gets an empty range (and is reported as invalid).
__global__ void k_surf_csr(const uint64_t* keys, int64_t nt, const int32_t* n_surf_p, int32_t* s_ptr, int32_t* s_tris,
                           int32_t* seen)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t n_surf = *n_surf_p;
    const int32_t s = i < nt ? (int32_t)(keys[i] >> 32) : 0;
    const int32_t prev = i == 0 ? -1 : i < nt ? (int32_t)(keys[i - 1] >> 32) : s;
    const unsigned long long heads = __ballot(i < nt && prev != s);
    if ((threadIdx.x & 63) == 0 && heads) atomicAdd(seen, (int)__popcll(heads));
    if (i >= nt) return;
    s_tris[i] = (int32_t)(keys[i] & 0xffffffffu);
    if (prev != s) {
        for (int32_t q = prev + 1; q <= s; ++q) s_ptr[q] = (int32_t)i;
    }
    if (i == nt - 1)
        for (int32_t q = s + 1; q <= n_surf; ++q) s_ptr[q] = (int32_t)nt;
}

// Tables of the surfaces, one wave per surface with the lanes over its
// triangles (one thread per surface, and per surface and grid cell, took 64 +
// 119 us for 1566 surfaces of 128 triangles; 13 us so).
//
// A surface's plane is that of its lowest-numbered triangle; every vertex of
// the surface must lie within RT_EPS (0.1 mm) of it (bad |= 16), and that
// triangle must not be degenerate (bad |= 32): the image method mirrors in
// this one plane for the whole surface.
//
// Containment grid: a surface gets one only if all its non-degenerate
// triangles use the same projection; a triangle is listed in every cell its
// projected box, grown by a margin that covers the rounding of the FP64 edge
// tests (relative to the coordinates and inversely to the shortest edge),
// overlaps.  Lists keep the surface's triangle order.
__device__ __forceinline__ double wave_dmin(double v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ double wave_dmax(double v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

__global__ __launch_bounds__(256) void k_surf_tables(const int32_t* s_ptr, const int32_t* s_tris, const double* v64,
                                                     const double* t_proj, const int32_t* t_axes,
                                                     const int32_t* n_surf_p, double* s_plane, double* s_box,
                                                     int32_t* g_axes, double* g_frame, int32_t* g_cnt,
                                                     int32_t* g_tris, int32_t* bad)
{
    const int lane = threadIdx.x & 63;
    const int n_surf = *n_surf_p;
    for (int s = (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)); s < n_surf;
         s += (int)(gridDim.x * (blockDim.x >> 6))) {
        const int b = s_ptr[s], e = s_ptr[s + 1];
        if (b >= e) {   // an unused id (reported as invalid)
            if (lane < 4) s_plane[4 * (int64_t)s + lane] = 0.0;
            if (lane < 6) s_box[6 * (int64_t)s + lane] = lane < 3 ? 1e300 : -1e300;
            if (lane == 0) g_axes[s] = -1;
            if (lane < RT_SGRID_CELLS) g_cnt[(int64_t)s * RT_SGRID_CELLS + lane] = 0;
            continue;
        }
        const double* v = v64 + 9 * (int64_t)s_tris[b];
        double e1[3], e2[3];
        for (int k = 0; k < 3; ++k) {
            e1[k] = v[3 + k] - v[k];
            e2[k] = v[6 + k] - v[k];
        }
        const double n0 = e1[1] * e2[2] - e1[2] * e2[1];
        const double n1 = e1[2] * e2[0] - e1[0] * e2[2];
        const double n2 = e1[0] * e2[1] - e1[1] * e2[0];
        const double dpl = n0 * v[0] + n1 * v[1] + n2 * v[2];
        const double nlen = sqrt(n0 * n0 + n1 * n1 + n2 * n2);
        const double tol = RT_EPS * nlen;
        bool off_plane = false;
        double lo[3] = {1e300, 1e300, 1e300}, hi[3] = {-1e300, -1e300, -1e300};
        int amin = 16, amax = -1;   // smallest and largest projection of the non-degenerate triangles
        for (int j = b + lane; j < e; j += 64) {
            const int t = s_tris[j];
            const double* w = v64 + 9 * (int64_t)t;
            for (int a = 0; a < 3; ++a) {
                for (int k = 0; k < 3; ++k) {
                    lo[k] = fmin(lo[k], w[3 * a + k]);
                    hi[k] = fmax(hi[k], w[3 * a + k]);
                }
                const double dist = n0 * w[3 * a] + n1 * w[3 * a + 1] + n2 * w[3 * a + 2] - dpl;
                off_plane |= !(fabs(dist) <= tol);
            }
            const int ax = t_axes[t];
            if (!(ax & 16)) {
                amin = min(amin, ax);
                amax = max(amax, ax);
            }
        }
        for (int k = 0; k < 3; ++k) {
            lo[k] = wave_dmin(lo[k]) - 1e-9;
            hi[k] = wave_dmax(hi[k]) + 1e-9;
        }
        amin = (int)wave_umin((unsigned)amin);
        amax = (int)wave_umax((unsigned)(amax + 1)) - 1;
        const bool any_off = __ballot(off_plane) != 0ull;
        if (lane == 0) {
            if (!(nlen > 0.0)) atomicOr(bad, 32);
            if (any_off) atomicOr(bad, 16);
            double* pl = s_plane + 4 * (int64_t)s;
            pl[0] = n0;
            pl[1] = n1;
            pl[2] = n2;
            pl[3] = dpl;
            for (int k = 0; k < 3; ++k) {
                s_box[6 * (int64_t)s + k] = lo[k];
                s_box[6 * (int64_t)s + 3 + k] = hi[k];
            }
        }
        const bool grid = amax >= 0 && amin == amax;
        const int i0 = grid ? amax & 3 : 0, i1 = grid ? (amax >> 2) & 3 : 1;
        const double u0 = i0 == 0 ? lo[0] : i0 == 1 ? lo[1] : lo[2], v0 = i1 == 0 ? lo[0] : i1 == 1 ? lo[1] : lo[2];
        const double eu = (i0 == 0 ? hi[0] : i0 == 1 ? hi[1] : hi[2]) - u0;
        const double ev = (i1 == 0 ? hi[0] : i1 == 1 ? hi[1] : hi[2]) - v0;
        const double pu = eu > 0.0 ? (double)RT_SGRID / eu : 0.0, pv = ev > 0.0 ? (double)RT_SGRID / ev : 0.0;
        if (lane == 0) {
            g_axes[s] = grid ? amax : -1;
            double* f = g_frame + 4 * (int64_t)s;
            f[0] = u0;
            f[1] = v0;
            f[2] = pu;
            f[3] = pv;
        }
        int cnt[RT_SGRID_CELLS];   // triangles listed so far per cell (the same on every lane)
#pragma unroll
        for (int c = 0; c < RT_SGRID_CELLS; ++c) cnt[c] = 0;
        const int64_t base = (int64_t)b * RT_SGRID_CELLS;
        for (int j0 = b; grid && j0 < e; j0 += 64) {
            unsigned cells = 0;   // bit per cell this lane's triangle goes to
            int t = -1;
            if (j0 + lane < e) {
                t = s_tris[j0 + lane];
                if (!(t_axes[t] & 16)) {   // a degenerate triangle contains nothing
                    const double* q = t_proj + 6 * (int64_t)t;
                    const double umin = fmin(q[0], fmin(q[2], q[4])), umax = fmax(q[0], fmax(q[2], q[4]));
                    const double vmin = fmin(q[1], fmin(q[3], q[5])), vmax = fmax(q[1], fmax(q[3], q[5]));
                    const double C = fmax(fmax(fabs(umin), fabs(umax)), fmax(fabs(vmin), fabs(vmax)));
                    const double l0 = hypot(q[2] - q[0], q[3] - q[1]), l1 = hypot(q[4] - q[2], q[5] - q[3]),
                                 l2 = hypot(q[0] - q[4], q[1] - q[5]);
                    const double lmin = fmax(fmin(l0, fmin(l1, l2)), 1e-300);
                    const double m = 1e-13 * (C * C / lmin) + 1e-9 * C + 1e-12;
                    const int c0 = sgrid_index(umin - m, u0, pu), c1 = sgrid_index(umax + m, u0, pu);
                    const int d0 = sgrid_index(vmin - m, v0, pv), d1 = sgrid_index(vmax + m, v0, pv);
                    const unsigned row = ((2u << d1) - 1u) & ~((1u << d0) - 1u);   // cells d0..d1 of one row
                    for (int i = c0; i <= c1; ++i) cells |= row << (RT_SGRID * i);
                }
            }
#pragma unroll
            for (int c = 0; c < RT_SGRID_CELLS; ++c) {
                const bool in = (cells >> c) & 1u;
                const unsigned long long m = __ballot(in);
                if (in) g_tris[base + (int64_t)c * (e - b) + cnt[c] + __popcll(m & ((1ull << lane) - 1ull))] = t;
                cnt[c] += (int)__popcll(m);
            }
        }
#pragma unroll
        for (int c = 0; c < RT_SGRID_CELLS; ++c)
            if (lane == c) g_cnt[(int64_t)s * RT_SGRID_CELLS + c] = cnt[c];
    }
}

static inline unsigned blocks_for(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

__global__ void k_ctl_init(unsigned* ctl)
{
    int i = threadIdx.x;
    if (i >= 64) return;
    unsigned v = 0u;
    if (i < 3 || (i >= 6 && i < 9)) v = 0xffffffffu;   // running minima
    ctl[i] = v;
}

// unit normal of e1 x e2 per triangle (0 for a degenerate triangle)
__global__ void k_unit_normals(const double* v64, int64_t nt, double* nrm)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nt) return;
    const double* v = v64 + 9 * t;
    const double ex = v[3] - v[0], ey = v[4] - v[1], ez = v[5] - v[2];
    const double fx = v[6] - v[0], fy = v[7] - v[1], fz = v[8] - v[2];
    const double nx = ey * fz - ez * fy, ny = ez * fx - ex * fz, nz = ex * fy - ey * fx;
    const double l = sqrt(nx * nx + ny * ny + nz * nz);
    const double il = l > 0.0 ? 1.0 / l : 0.0;
    nrm[3 * t + 0] = nx * il;
    nrm[3 * t + 1] = ny * il;
    nrm[3 * t + 2] = nz * il;
}

void scene_normals(Ctx& c, Scene& s, hipStream_t st)
{
    if (s.n_tri == 0 || s.nrm.bytes) return;
    s.nrm = Scratch(c, sizeof(double) * 3 * (size_t)s.n_tri, st);
    hipLaunchKernelGGL(k_unit_normals, dim3(blocks_for(s.n_tri, 256)), dim3(256), 0, st, s.v64.as<double>(), s.n_tri,
                       s.nrm.as<double>());
    HIP_CHECK(hipGetLastError());
}

void build_scene(Ctx& c, Scene& s, const float* V, int64_t nv, const int32_t* T, int64_t nt,
                 const int32_t* surf, const float* rr, const float* ri, hipStream_t st)
{
    s.n_tri = nt;
    if (nt == 0) {
        s.n_surf = 0;
        s.root = 0;
        return;
    }
    if (nt >= (int64_t)1 << 29) throw inval_error("too many triangles (at most 2^29 - 1)");
    // inputs in device memory are read in place (the build is complete before the call returns);
    // host arrays are staged
    Scratch stage_buf[5];
    auto input = [&](const void* p, size_t bytes, int slot) -> const void* {
        if (bytes == 0 || is_device_ptr(p)) return p;
        stage_buf[slot] = Scratch(c, bytes, st);
        HIP_CHECK(hipMemcpyAsync(stage_buf[slot].p, p, bytes, hipMemcpyDefault, st));
        return stage_buf[slot].p;
    };
    const float* dV = (const float*)input(V, sizeof(float) * 3 * (size_t)nv, 0);
    const int32_t* dT = (const int32_t*)input(T, sizeof(int32_t) * 3 * (size_t)nt, 1);
    const int32_t* dS = (const int32_t*)input(surf, sizeof(int32_t) * (size_t)nt, 2);
    const float* dR = (const float*)input(rr, sizeof(float) * (size_t)nt, 3);
    const float* dI = (const float*)input(ri, sizeof(float) * (size_t)nt, 4);

    s.v64 = Scratch(c, sizeof(double) * 9 * (size_t)nt, st);
    s.t_proj = Scratch(c, sizeof(double) * 6 * (size_t)nt, st);
    s.t_axes = Scratch(c, sizeof(int32_t) * (size_t)nt, st);
    s.refl = Scratch(c, sizeof(float2) * (size_t)nt, st);
    s.surf = Scratch(c, sizeof(int32_t) * (size_t)nt, st);
    s.tri4 = Scratch(c, sizeof(float4) * 3 * (size_t)nt, st);
    Scratch cent(c, sizeof(float4) * (size_t)nt, st);
    // control block: bounds[12] unsigned, bad, maxdepth, n_surf, seen, nodes spanning several refit tiles
    Scratch ctl(c, 64 * sizeof(int32_t), st);
    unsigned* bounds = ctl.as<unsigned>();
    int32_t* bad = ctl.as<int32_t>() + 12;
    int32_t* maxd = ctl.as<int32_t>() + 13;
    int32_t* nsurf = ctl.as<int32_t>() + 14;
    int32_t* seen = ctl.as<int32_t>() + 15;
    int32_t* ncross = ctl.as<int32_t>() + 16;
    hipLaunchKernelGGL(k_ctl_init, dim3(1), dim3(64), 0, st, bounds);
    HIP_CHECK(hipGetLastError());
    const int B = 256;
    Scratch skeys(c, sizeof(uint64_t) * (size_t)nt, st);
    hipLaunchKernelGGL(k_scene_prep, dim3(std::min<unsigned>(blocks_for(nt, PREP_B), PREP_BLOCKS)), dim3(PREP_B), 0, st,
                       dV, dT, dS, dR, dI, nv, nt, s.v64.as<double>(), s.refl.as<float2>(), s.surf.as<int32_t>(),
                       cent.as<float4>(), skeys.as<uint64_t>(), bounds, bad, nsurf, s.t_proj.as<double>(),
                       s.t_axes.as<int32_t>());
    HIP_CHECK(hipGetLastError());
    s.box = Scratch(c, 6 * sizeof(float), st);
    Scratch keys_raw(c, 2 * sizeof(uint64_t) * (size_t)nt, st), keys(c, 2 * sizeof(uint64_t) * (size_t)nt, st);
    hipLaunchKernelGGL(k_morton, dim3(blocks_for(nt, B)), dim3(B), 0, st, cent.as<float4>(), bounds, nt,
                       keys_raw.as<uint64_t>(), s.box.as<float>());
    HIP_CHECK(hipGetLastError());
    sort_keys(c, keys_raw.as<uint64_t>(), keys.as<uint64_t>(), nt, 2, 64, 127, st);
    Scratch lbox(c, sizeof(float) * 6 * (size_t)nt, st);
    hipLaunchKernelGGL(k_leaves, dim3(blocks_for(nt, B)), dim3(B), 0, st, keys.as<uint64_t>(), dV, dT,
                       s.surf.as<int32_t>(), nv, nt, bounds, s.tri4.as<float4>(), lbox.as<float>());
    HIP_CHECK(hipGetLastError());

    if (nt >= 2) {
        int64_t ni = nt - 1;
        s.nodes = Scratch(c, sizeof(float4) * 4 * (size_t)ni, st);
        const int64_t n_tiles = (nt + RT_REFIT_TILE - 1) / RT_REFIT_TILE;
        Scratch child(c, sizeof(int32_t) * 2 * (size_t)ni, st), pint(c, sizeof(int32_t) * (size_t)ni, st),
            pleaf(c, sizeof(int32_t) * (size_t)nt, st), range(c, sizeof(int2) * (size_t)ni, st),
            cross(c, sizeof(int32_t) * (size_t)(n_tiles > 1 ? ni : 1), st),
            tbox(c, sizeof(float) * 6 * (size_t)n_tiles, st);
        hipLaunchKernelGGL(k_karras, dim3(blocks_for(ni, B)), dim3(B), 0, st, keys.as<uint64_t>(), nt,
                           child.as<int32_t>(), pint.as<int32_t>(), pleaf.as<int32_t>(), range.as<int2>(),
                           cross.as<int32_t>(), ncross);
        HIP_CHECK(hipGetLastError());
        hipLaunchKernelGGL(k_refit_tiles, dim3((unsigned)n_tiles), dim3(1024), 0, st, child.as<int32_t>(),
                           pint.as<int32_t>(), pleaf.as<int32_t>(), range.as<int2>(), lbox.as<float>(),
                           s.nodes.as<float4>(), nt, tbox.as<float>(), bad);
        HIP_CHECK(hipGetLastError());
        if (n_tiles > 1) {
            hipLaunchKernelGGL(k_refit_cross, dim3(512), dim3(256), 0, st, cross.as<int32_t>(), ncross,
                               child.as<int32_t>(), pint.as<int32_t>(), pleaf.as<int32_t>(), range.as<int2>(),
                               lbox.as<float>(), tbox.as<float>(), s.nodes.as<float4>(), bad);
            HIP_CHECK(hipGetLastError());
        }
        s.node4 = Scratch(c, sizeof(float4) * 8 * (size_t)ni, st);
        hipLaunchKernelGGL(k_node4, dim3(blocks_for(ni, B)), dim3(B), 0, st, child.as<int32_t>(), pint.as<int32_t>(),
                           s.nodes.as<float4>(), s.tri4.as<float4>(), ni, s.node4.as<float4>(), maxd);
        HIP_CHECK(hipGetLastError());
        s.root = 0;
    } else {
        s.root = ~0;
    }

    // surfaces (tables sized for the largest valid count, n_surf <= n_tri)
    {
        // the keys come in triangle order and the sort is stable: the surface bits decide alone
        int sbits = 1;
        while (((int64_t)1 << sbits) < nt) ++sbits;
        Scratch sorted(c, sizeof(uint64_t) * (size_t)nt, st);
        sort_keys(c, skeys.as<uint64_t>(), sorted.as<uint64_t>(), nt, 1, 32, 32 + sbits, st);
        std::swap(skeys, sorted);
    }
    s.s_ptr = Scratch(c, sizeof(int32_t) * (size_t)(nt + 1), st);
    s.s_tris = Scratch(c, sizeof(int32_t) * (size_t)nt, st);
    s.s_plane = Scratch(c, sizeof(double) * 4 * (size_t)nt, st);
    s.s_box = Scratch(c, sizeof(double) * 6 * (size_t)nt, st);
    hipLaunchKernelGGL(k_surf_csr, dim3(blocks_for(nt, B)), dim3(B), 0, st, skeys.as<uint64_t>(), nt, nsurf,
                       s.s_ptr.as<int32_t>(), s.s_tris.as<int32_t>(), seen);
    HIP_CHECK(hipGetLastError());
    s.g_axes = Scratch(c, sizeof(int32_t) * (size_t)nt, st);
    s.g_frame = Scratch(c, sizeof(double) * 4 * (size_t)nt, st);
    s.g_cnt = Scratch(c, sizeof(int32_t) * RT_SGRID_CELLS * (size_t)nt, st);
    s.g_tris = Scratch(c, sizeof(int32_t) * RT_SGRID_CELLS * (size_t)nt, st);
    hipLaunchKernelGGL(k_surf_tables, dim3(std::min<unsigned>(blocks_for(nt, 4), 2048)), dim3(256), 0, st,
                       s.s_ptr.as<int32_t>(), s.s_tris.as<int32_t>(), s.v64.as<double>(), s.t_proj.as<double>(),
                       s.t_axes.as<int32_t>(), nsurf, s.s_plane.as<double>(), s.s_box.as<double>(),
                       s.g_axes.as<int32_t>(), s.g_frame.as<double>(), s.g_cnt.as<int32_t>(),
                       s.g_tris.as<int32_t>(), bad);
    HIP_CHECK(hipGetLastError());
    // one read-back: input checks, tree checks, surface count
    int64_t hq[2];
    read_i64s((const int64_t*)(ctl.as<int32_t>() + 12), hq, 2, st);
    const int32_t badv = (int32_t)(hq[0] & 0xffffffff), depth = (int32_t)(hq[0] >> 32);
    const int32_t n_surf = (int32_t)(hq[1] & 0xffffffff), n_seen = (int32_t)(hq[1] >> 32);
    if (badv & 1) throw inval_error("triangle vertex index out of range");
    if (badv & 2) throw inval_error("vertex coordinate not finite or |x| > 1e6");
    if (badv & 4) throw inval_error("surface id outside 0..n_tri-1");
    if (badv & 8) throw hip_error("BVH build produced an inconsistent tree");
    if (depth > RT_STACK - 1) throw inval_error("BVH deeper than the traversal stack");
    if (n_seen != n_surf) throw inval_error("surface ids must be 0..n_surf-1, each used");
    if (n_surf > (1 << RT_KEY_BITS) - 1)   // a candidate key holds surface id + 1 in 21 bits
        throw inval_error("at most 2^21 - 1 surfaces");
    if (badv & 32) throw inval_error("the lowest-numbered triangle of a surface is degenerate (no plane)");
    if (badv & 16) throw inval_error("the triangles of a surface are not coplanar (a vertex lies more than "
                                     "0.1 mm from the plane of the surface's first triangle)");
    s.max_depth = depth;
    s.n_surf = n_surf;
}

}  // namespace rt
