// Scene upload and BVH build on the device.
//
// Two trees over the same leaves:
//
//  * The linear BVH after Karras, "Maximizing Parallelism in the Construction
//    of BVHs, Octrees, and k-d Trees" (HPG 2012): 63-bit Morton codes of
//    triangle centroids with the triangle index as tie-break, radix sort, one
//    thread per internal node finds its key range and split.  Its depth is the
//    one a scene reports and is limited by, and the counting builds walk it
//    (lbvh_nodes gives it its boxes then).
//  * The tree every other walk takes: a linear BVH of each surface's triangles
//    (Morton order within the surface), and above the surfaces' subtrees a
//    binned surface-area split of their boxes.  Triangles of one surface are
//    coplanar, so its subtree's boxes are flat, while a Morton order over the
//    whole scene mixes triangles of different faces in one box: half the nodes
//    visited (lab room: 41 -> 24 in relative box area, a wave of discovery rays
//    visits 11 instead of 19 four-wide nodes per bounce, the path kernels run
//    239 + 201 instead of 397 + 387 us; office floor 188 -> 99, 41 -> 26,
//    discovery 8.6 + 11.6 instead of 11.4 + 15.8 ms).  Scenes of more than RT_TOP_MAX surfaces (the split runs in one
//    workgroup), or where that tree came out deeper than the traversal stacks
//    hold, take the linear BVH of the whole scene for it.
//
// Node boxes are computed bottom-up within tiles of leaves and by leaf range
// above them, and are inflated so that the FP32 slab test is conservative with
// respect to the exact ray/triangle formula.
//
// Layouts (leaf slot = rank of the triangle by surface, then Morton code):
//   tri4  [3 * n]: (v0.xyz, id), (e1.xyz, surface), (e2.xyz, 0)
//   nodes [4 * ..]: (loL.xyz, childL), (hiL.xyz, childR), (loR.xyz, -), (hiR.xyz, -)
//   child >= 0: internal node; child < 0: leaf slot ~child.  Node indices are
//   those of the Karras nodes over the slots; the nodes above the surfaces take
//   the indices of the Karras nodes that span several surfaces.
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

// Vertices per triangle, edge functions, reflection coefficients, surface
// ids and sort keys (surface above triangle), centroids; bounds of the
// centroids and of the vertices (order-preserving unsigned keys) and the
// largest surface id.  Every block ends in 13 atomics on the same few words,
// which serialise across the XCDs: at most PREP_BLOCKS blocks stride over the
// triangles and reduce in LDS first (200 000 triangles: 444 us with 12 atomics
// per wave, 30 us so).
constexpr int PREP_B = 256, PREP_BLOCKS = 512;
__global__ __launch_bounds__(PREP_B) void k_scene_prep(const float* V, const int32_t* T, const int32_t* surf_in,
                                                       const float* rr, const float* ri, int64_t nv, int64_t nt,
                                                       float* verts, float2* refl, int32_t* surf, float4* cent,
                                                       uint64_t* skeys, unsigned* bounds, int32_t* bad,
                                                       int32_t* n_surf, double* edge)
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
                verts[9 * t + 3 * j + k] = x;
                c[k] += x;
                const unsigned u = f2ord(x);
                mn[3 + k] = min(mn[3 + k], u);
                mx[3 + k] = max(mx[3 + k], u);
            }
        }
        double q6[6];
        int32_t ax;
        triangle_projection(w, q6, &ax);
        triangle_edges(q6, ax, edge + RT_EDGE * t);
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

// Keys of the leaf slots from the triangles in Morton order: word 1 surface
// (21 bits) above the code's upper 43 bits, word 0 its lower 20 bits above the
// triangle index (29 bits).  Sorted stably on the surface bits alone.  Without
// surfaces above the Morton order (plain, or too many of them) they are all 0.
constexpr uint64_t RT_KEY_TRI = (1ull << 29) - 1;
constexpr int RT_KEY_SURF_SHIFT = 43;   // in word 1
__global__ void k_slot_keys(const uint64_t* keys, const int32_t* surf, int64_t nt, const int32_t* n_surf_p, int plain,
                            uint64_t* out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nt) return;
    const uint64_t t = keys[2 * i], code = keys[2 * i + 1];
    const int32_t sf = surf[t];
    const uint64_t sc = plain || !top_wanted(*n_surf_p) ? 0ull : (uint64_t)(sf < 0 ? 0 : (sf >= nt ? nt - 1 : sf));
    out[2 * i] = ((code & 0xfffffull) << 29) | t;
    out[2 * i + 1] = (sc << RT_KEY_SURF_SHIFT) | (code >> 20);
}

// Is there a tree above the surfaces' subtrees?  (Every id used: an unused one
// is reported after the build.)
__device__ __forceinline__ bool top_used(int n_surf, int seen)
{
    return top_wanted(n_surf) && seen == n_surf;
}

__device__ __forceinline__ int64_t clamp_index(int32_t v, int64_t n) { return v < 0 ? 0 : (v >= n ? n - 1 : v); }

// Leaf data in sorted order.  Box padding: 1e-5 of the scene extent + 1e-6 m
// + 1e-5 |x| (indices are clamped: malformed input is reported after the build).
__global__ void k_leaves(const uint64_t* keys, const float* V, const int32_t* T, const int32_t* surf, int64_t nv,
                         int64_t nt, const unsigned* bounds, float4* tri4, float* lbox, int32_t* tslot)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nt) return;
    float ext = 0.0f;
    for (int k = 0; k < 3; ++k) ext = fmaxf(ext, ord2f(bounds[9 + k]) - ord2f(bounds[6 + k]));
    const float pad = 1e-5f * ext + 1e-6f;
    const int32_t t = (int32_t)(keys[2 * i] & RT_KEY_TRI);   // low bits of word 0: the triangle index
    tslot[t] = (int32_t)i;
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

// One thread per internal node and tree (blockIdx.y 0: the slots' tree, 1: the
// scene's Morton tree): children and parent links; for the slots' tree also the
// leaf range below the node, and the nodes whose leaves span several refit
// tiles are listed (in no fixed order) for k_refit_cross.
struct KarrasOut {
    const uint64_t* keys;
    int32_t* child;
    int32_t* parent_int;
    int32_t* parent_leaf;
};
__global__ void k_karras(KarrasOut slots, KarrasOut morton, int64_t n, int2* range, int32_t* cross, int32_t* n_cross)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n - 1) return;
    const KarrasOut o = blockIdx.y == 0 ? slots : morton;
    if (i == 0) o.parent_int[0] = -1;   // the root; every other node and every leaf gets its parent below
    int32_t cl, cr, first, last;
    lbvh_node<2>(o.keys, n, i, &cl, &cr, &first, &last);
    if (cl >= 0) o.parent_int[cl] = (int32_t)i;
    if (cr >= 0) o.parent_int[cr] = (int32_t)i;
    o.child[2 * i] = cl;
    o.child[2 * i + 1] = cr;
    if (blockIdx.y != 0) return;
    if (cl < 0) o.parent_leaf[~cl] = (int32_t)i;
    if (cr < 0) o.parent_leaf[~cr] = (int32_t)i;
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

// --------------------------------------------------------------------------
// The tree above the surfaces: binned surface-area splits (Wald, "On fast
// Construction of SAH-based Bounding Volume Hierarchies", RT 2007: bins along
// the centroids' extent, cost = area x triangles on either side).  A wave
// takes a range of surfaces: lane l weighs the split q % 10 + 1 of TOP_BINS
// bins along axis q / 10, q = l % 32 (30 of 32 lanes), the two halves of the
// wave take alternate surfaces, so one pass over the range prices all 30
// splits with no atomics and no bin memory.  The work is small and serial
// (about 20 instructions per surface and level, then a chain of reductions
// per node), so what bounds it is latency: the boxes stay in LDS where they
// fit (up to TOP_RES surfaces).  Ranges are split level by level in one
// workgroup, large ones by all its waves together: up to TOP_LEAF surfaces to
// the end, beyond until they hold at most TOP_LEAF, and those go one workgroup
// each over the device: 106 surfaces 67 us, 1566 surfaces 175 + 116 us.  The
// boxes of more surfaces than TOP_RES are gathered from memory at every level
// (8192 surfaces 1074 + 138 us), so where surfaces are many and have few
// triangles (top_full) the upper levels split groups of them instead: TOP_GROUP
// consecutive ones along a Morton order, each group by a workgroup of its own
// (8000 surfaces 220 us in all instead of 990, traces of 10^5 rays 800 instead of 774
// us; 969 without a split).
// Of the n Karras indices 0..n-1 over the slots (n - 1 is no node), a surface's
// c triangles hold c, its subtree takes c - 1 of them and leaves one end free:
// the index of a Karras node over several surfaces (the last surface leaves
// n - 1).  A range split before position m takes the one that surface m - 1
// left (every position splits once), so the numbering needs neither a counter
// nor room of its own.
// --------------------------------------------------------------------------
constexpr int TOP_BINS = 11, TOP_LEAF = 256, TOP_T = 1024, TOP_RES = RT_TOP_RES, TOP_FT = 512, TOP_GROUP = 64;
constexpr int TOP_Q = TOP_LEAF / 2;   // ranges of a level: of two surfaces (or groups) and more, or of more than TOP_LEAF
static_assert(RT_TOP_MAX / (TOP_LEAF + 1) <= TOP_Q && RT_TOP_MAX / TOP_GROUP / 2 <= TOP_Q, "a level's ranges fit the queue");

struct TopOut {
    float4* nodes;
    int32_t* child;
    int32_t* parent_int;
    int32_t* root;
    const int32_t* ids;   // node index of split position 1, 2, ...
};

// child `ref` of side `side` of node `parent` (-1: the root)
__device__ __forceinline__ void top_link(const TopOut& o, int parent, int side, int ref)
{
    if (parent < 0) {
        *o.root = ref;
    } else {
        o.child[2 * (int64_t)parent + side] = ref;
        ((int32_t*)o.nodes)[16 * (int64_t)parent + 4 * side + 3] = ref;
    }
    if (ref >= 0) o.parent_int[ref] = parent;
}

// The surfaces' boxes as two float4 each: lo.xyz and the triangle count, hi.xyz
// and the subtree's reference (in LDS or global memory; the functions that take
// them are inlined, so each use has its own kind of load).
struct TopBoxes {
    const float4* p;
    __device__ __forceinline__ float4 get(int i) const { return p[i]; }
};

// one lane's price of its split: boxes and triangle counts left and right
struct TopAcc {
    float l[6], r[6], wl, wr;
};
__device__ __forceinline__ void top_clear(TopAcc& a)
{
    for (int k = 0; k < 3; ++k) {
        a.l[k] = a.r[k] = 3e38f;
        a.l[3 + k] = a.r[3 + k] = -3e38f;
    }
    a.wl = a.wr = 0.0f;
}
__device__ __forceinline__ void top_merge(TopAcc& a, const TopAcc& b)
{
    for (int k = 0; k < 3; ++k) {
        a.l[k] = fminf(a.l[k], b.l[k]);
        a.r[k] = fminf(a.r[k], b.r[k]);
        a.l[3 + k] = fmaxf(a.l[3 + k], b.l[3 + k]);
        a.r[3 + k] = fmaxf(a.r[3 + k], b.r[3 + k]);
    }
    a.wl += b.wl;
    a.wr += b.wr;
}
// the other half of the wave's prices of the same splits
__device__ __forceinline__ void top_merge_halves(TopAcc& a)
{
    TopAcc o;
    for (int k = 0; k < 6; ++k) {
        o.l[k] = __shfl_xor(a.l[k], 32, 64);
        o.r[k] = __shfl_xor(a.r[k], 32, 64);
    }
    o.wl = __shfl_xor(a.wl, 32, 64);
    o.wr = __shfl_xor(a.wr, 32, 64);
    top_merge(a, o);
}
// Bin coordinate of a box along an axis: left of split s if below s.  `c`: the
// extent of the doubled centres, three minima, three maxima.
struct TopAxis {
    int axis;
    float c0, scale;
    __device__ __forceinline__ TopAxis(int a, const float* c) : axis(a)
    {
        c0 = a == 0 ? c[0] : a == 1 ? c[1] : c[2];
        const float ext = (a == 0 ? c[3] : a == 1 ? c[4] : c[5]) - c0;
        scale = ext > 0.0f ? (float)TOP_BINS / ext : 0.0f;
    }
    __device__ __forceinline__ float bin(float4 lo, float4 hi) const
    {
        const float v = axis == 0 ? lo.x + hi.x : axis == 1 ? lo.y + hi.y : lo.z + hi.z;
        return (v - c0) * scale;
    }
};

// extent of the doubled centres over positions first, first + step, ... below b of every lane
__device__ __forceinline__ void top_extent(const TopBoxes sb, const uint16_t* idx, int first, int b, int step, float* c)
{
    for (int k = 0; k < 3; ++k) {
        c[k] = 3e38f;
        c[3 + k] = -3e38f;
    }
    for (int i = first; i < b; i += step) {
        const int s = idx[i];
        const float4 lo = sb.get(2 * s), hi = sb.get(2 * s + 1);
        const float v[3] = {lo.x + hi.x, lo.y + hi.y, lo.z + hi.z};
        for (int k = 0; k < 3; ++k) {
            c[k] = fminf(c[k], v[k]);
            c[3 + k] = fmaxf(c[3 + k], v[k]);
        }
    }
    for (int k = 0; k < 3; ++k) {
        c[k] = -wave_max(-c[k]);
        c[3 + k] = wave_max(c[3 + k]);
    }
}

// every lane's price of its split over positions [a, b) in chunks of 64 taken `stride` apart
__device__ __forceinline__ void top_price(const TopBoxes sb, const uint16_t* idx, int a, int b, int stride,
                                          const float* c, TopAcc& acc)
{
    const int lane = threadIdx.x & 63, q = lane & 31, half = lane >> 5;
    const TopAxis ax(min(q / 10, 2), c);
    const float split = (float)(q % 10 + 1);
    top_clear(acc);
    for (int i0 = a; i0 < b; i0 += stride) {
        const int n = min(64, b - i0);
        // eight surfaces at a time, their reads in flight together (past the end: the last one, counted nowhere)
        for (int j0 = half; j0 < n; j0 += 8) {
            float4 lo[4], hi[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int s = idx[i0 + min(j0 + 2 * u, n - 1)];
                lo[u] = sb.get(2 * s);
                hi[u] = sb.get(2 * s + 1);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool in = j0 + 2 * u < n, below = ax.bin(lo[u], hi[u]) < split;
                const bool left = in && below, right = in && !below;
                const float m[6] = {lo[u].x, lo[u].y, lo[u].z, hi[u].x, hi[u].y, hi[u].z};
                for (int k = 0; k < 3; ++k) {
                    acc.l[k] = fminf(acc.l[k], left ? m[k] : 3e38f);
                    acc.r[k] = fminf(acc.r[k], right ? m[k] : 3e38f);
                    acc.l[3 + k] = fmaxf(acc.l[3 + k], left ? m[3 + k] : -3e38f);
                    acc.r[3 + k] = fmaxf(acc.r[3 + k], right ? m[3 + k] : -3e38f);
                }
                acc.wl += left ? lo[u].w : 0.0f;
                acc.wr += right ? lo[u].w : 0.0f;
            }
        }
    }
}

// the node of split position m: its children's boxes and its link (lane 0)
__device__ __forceinline__ void top_node(const TopOut& o, int m, int parent, int side, const float* l, const float* r)
{
    if ((threadIdx.x & 63) != 0) return;
    const int id = o.ids[m - 1];
    float* nd = (float*)(o.nodes + 4 * (int64_t)id);   // the .w words are links
    for (int k = 0; k < 3; ++k) {
        nd[k] = l[k];
        nd[4 + k] = l[3 + k];
        nd[8 + k] = r[k];
        nd[12 + k] = r[3 + k];
    }
    nd[11] = nd[15] = 0.0f;
    top_link(o, parent, side, id);
}

// A range of two surfaces (about a third of all ranges): nothing to choose.
template <class Single>
__device__ __forceinline__ void top_pair(const TopBoxes sb, const uint16_t* idx, int a, int parent, int side,
                                         const TopOut& o, Single single)
{
    const int s0 = idx[a], s1 = idx[a + 1];
    const float4 l0 = sb.get(2 * s0), h0 = sb.get(2 * s0 + 1), l1 = sb.get(2 * s1), h1 = sb.get(2 * s1 + 1);
    const float l[6] = {l0.x, l0.y, l0.z, h0.x, h0.y, h0.z}, r[6] = {l1.x, l1.y, l1.z, h1.x, h1.y, h1.z};
    top_node(o, a + 1, parent, side, l, r);
    if ((threadIdx.x & 63) == 0) {
        const int id = o.ids[a];
        single(s0, id, 0);
        single(s1, id, 1);
    }
}

// One range [a, b) from its prices (halves merged): choose the cheapest split,
// partition idx stably, write the node's boxes and its link.  Returns the
// split position (strictly inside; the middle where no split has surfaces on
// both sides).  All lanes of one wave.
__device__ __forceinline__ int top_split(const TopBoxes sb, uint16_t* idx, uint16_t* tmp, int a, int b, int parent,
                                         int side, const float* c, const TopAcc& acc, const TopOut& o)
{
    const int lane = threadIdx.x & 63, q = lane & 31;
    auto area = [](const float* m) {
        const float x = m[3] - m[0], y = m[4] - m[1], z = m[5] - m[2];
        return x * y + y * z + z * x;
    };
    const float none = 3e38f;
    float cost = q < 30 && acc.wl > 0.0f && acc.wr > 0.0f ? area(acc.l) * acc.wl + area(acc.r) * acc.wr : none;
    if (!(cost < none)) cost = none;
    const float best = -wave_max(-cost);
    const bool by_price = best < none;
    const int who = __ffsll((long long)__ballot(cost == best)) - 1;   // ties: the first split
    const TopAxis ax(min((who & 31) / 10, 2), c);
    const float split = (float)((who & 31) % 10 + 1);
    int m = a + (b - a) / 2;
    float l[6], r[6];
    if (by_price) {
        // stable partition: lefts move down in place, rights wait in tmp (the same positions, so that
        // ranges split at the same time do not meet)
        int nl = 0, nr = 0;
        for (int i0 = a; i0 < b; i0 += 64) {
            const bool in = i0 + lane < b;
            const uint16_t s = in ? idx[i0 + lane] : (uint16_t)0;
            const bool left = in && ax.bin(sb.get(2 * s), sb.get(2 * s + 1)) < split;
            const unsigned long long ml = __ballot(left), mr = __ballot(in && !left);
            const unsigned long long lt = (1ull << lane) - 1ull;
            if (left) idx[a + nl + __popcll(ml & lt)] = s;
            if (in && !left) tmp[a + nr + __popcll(mr & lt)] = s;
            nl += (int)__popcll(ml);
            nr += (int)__popcll(mr);
        }
        m = a + nl;
        for (int i = lane; i < nr; i += 64) idx[m + i] = tmp[a + i];
        for (int k = 0; k < 6; ++k) {
            l[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(acc.l[k]), who));
            r[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(acc.r[k]), who));
        }
    } else {
        TopAcc t;
        top_clear(t);
        for (int i = a + lane; i < b; i += 64) {
            const int s = idx[i];
            const float4 lo = sb.get(2 * s), hi = sb.get(2 * s + 1);
            const bool left = i < m;
            const float v[6] = {lo.x, lo.y, lo.z, hi.x, hi.y, hi.z};
            for (int k = 0; k < 3; ++k) {
                t.l[k] = fminf(t.l[k], left ? v[k] : 3e38f);
                t.r[k] = fminf(t.r[k], left ? 3e38f : v[k]);
                t.l[3 + k] = fmaxf(t.l[3 + k], left ? v[3 + k] : -3e38f);
                t.r[3 + k] = fmaxf(t.r[3 + k], left ? -3e38f : v[3 + k]);
            }
        }
        for (int k = 0; k < 3; ++k) {
            l[k] = -wave_max(-t.l[k]);
            r[k] = -wave_max(-t.r[k]);
            l[3 + k] = wave_max(t.l[3 + k]);
            r[3 + k] = wave_max(t.r[3 + k]);
        }
    }
    top_node(o, m, parent, side, l, r);
    return m;
}

// A workgroup's shared state: up to CAP surfaces, the boxes of RES, T threads.
template <int CAP, int RES, int T, int Q>
struct TopShared {
    static constexpr int NW = T / 64, MAX = CAP;
    alignas(16) uint16_t idx[CAP];
    uint16_t tmp[CAP];
    int32_t ids[RES];
    float4 box[2 * RES];
    TopAcc part[NW][32];
    float ext[NW][6];
    int4 queue[2][Q];
    int nq[2], nfin;
};

// A barrier that orders LDS alone: the nodes written to memory are not read again here, and waiting for those
// stores at every level would cost more than the level.
__device__ __forceinline__ void top_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Where group g of n_group of n surfaces begins (and the one before it ends).
__device__ __forceinline__ int top_group(int g, int n_group, int n) { return (int)((int64_t)g * n / n_group); }

// The range in queue[0], of n_item in all, split level by level until its parts hold at most `leaf` surfaces.
// n_group > 0: what is split are that many groups of n surfaces, and a single one goes to fin.
template <class Shared>
__device__ __forceinline__ void top_levels(Shared& sh, const TopBoxes sb, int n_item, int leaf, int n_group, int n,
                                           int4* fin, const TopOut& o)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    constexpr int NW = Shared::NW, T = NW * 64;
    auto single = [&](int item, int parent, int side) {
        if (n_group > 0)
            fin[atomicAdd(&sh.nfin, 1)] =
                make_int4(top_group(item, n_group, n), top_group(item + 1, n_group, n), parent, side);
        else
            top_link(o, parent, side, __float_as_int(sb.get(2 * item + 1).w));
    };
    // a part of a split range: split again, left to a workgroup, or one surface (its link) or group
    auto hand_on = [&](int a, int b, int parent, int side, int to) {
        if (b - a == 1)
            single(sh.idx[a], parent, side);
        else if (b - a > leaf)
            sh.queue[to][atomicAdd(&sh.nq[to], 1)] = make_int4(a, b, parent, side);
        else
            fin[atomicAdd(&sh.nfin, 1)] = make_int4(a, b, parent, side);
    };
    for (int cur = 0;; cur ^= 1) {
        const int cnt = sh.nq[cur];
        if (cnt == 0) break;
        // few ranges: all waves price each together
        const bool together = cnt <= 4 && n_item > 128 * cnt;
        for (int e = together ? 0 : wave; e < cnt; e += together ? 1 : NW) {
            const int4 it = sh.queue[cur][e];
            if (it.y - it.x == 2) {
                if (!together || wave == 0) top_pair(sb, sh.idx, it.x, it.z, it.w, o, single);
                continue;
            }
            // one copy of the code for both (a cold instruction cache costs more than the arithmetic)
            float c[6];
            TopAcc acc;
            top_extent(sb, sh.idx, it.x + (together ? (int)threadIdx.x : lane), it.y, together ? T : 64, c);
            if (together) {
                if (lane == 0)
                    for (int k = 0; k < 6; ++k) sh.ext[wave][k] = c[k];
                top_barrier();
#pragma unroll 1
                for (int w = 0; w < NW; ++w)
                    for (int k = 0; k < 3; ++k) {
                        c[k] = fminf(c[k], sh.ext[w][k]);
                        c[3 + k] = fmaxf(c[3 + k], sh.ext[w][3 + k]);
                    }
            }
            top_price(sb, sh.idx, it.x + (together ? 64 * wave : 0), it.y, together ? T : 64, c, acc);
            top_merge_halves(acc);
            if (together) {
                if (lane < 32) sh.part[wave][lane] = acc;
                top_barrier();
                if (wave == 0) {
#pragma unroll 1
                    for (int w = 1; w < NW; ++w) top_merge(acc, sh.part[w][lane & 31]);
                }
            }
            if (!together || wave == 0) {
                const int m = top_split(sb, sh.idx, sh.tmp, it.x, it.y, it.z, it.w, c, acc, o);
                if (lane == 0) {
                    const int id = o.ids[m - 1];
                    hand_on(it.x, m, id, 0, cur ^ 1);
                    hand_on(m, it.y, id, 1, cur ^ 1);
                }
            }
            if (together) top_barrier();
        }
        top_barrier();
        if (threadIdx.x == 0) sh.nq[cur] = 0;
        top_barrier();
    }
}

// Surfaces in Morton order of their boxes' centres (a bitonic sort in LDS, in
// the room of sh.idx and sh.tmp), and the boxes, triangle counts and node
// indices of the n_group groups of them.  ce: this thread's extent of the
// doubled centres.
template <class Shared>
__device__ __forceinline__ void top_groups(Shared& sh, int n, int n_group, float* ce, const float4* sb,
                                           const int32_t* ids, int32_t* order_out)
{
    const int tid = (int)threadIdx.x, wave = tid >> 6, lane = tid & 63;
    constexpr int NW = Shared::NW, T = NW * 64;
    static_assert(Shared::MAX >= RT_TOP_MAX && RT_TOP_MAX <= 1 << 13, "room for a key a surface, 13 bits for a surface");
    uint32_t* keys = (uint32_t*)sh.idx;   // Morton code, 6 bits an axis, above the surface
    for (int k = 0; k < 3; ++k) {
        ce[k] = -wave_max(-ce[k]);
        ce[3 + k] = wave_max(ce[3 + k]);
    }
    if (lane == 0)
        for (int k = 0; k < 6; ++k) sh.ext[wave][k] = ce[k];
    __syncthreads();   // the boxes in sb too
    for (int w = 0; w < NW; ++w)
        for (int k = 0; k < 3; ++k) {
            ce[k] = fminf(ce[k], sh.ext[w][k]);
            ce[3 + k] = fmaxf(ce[3 + k], sh.ext[w][3 + k]);
        }
    int n2 = 2;
    while (n2 < n) n2 <<= 1;
    for (int s = tid; s < n2; s += T) {
        uint32_t key = 0xffffffffu;
        if (s < n) {
            const float4 lo = sb[2 * s], hi = sb[2 * s + 1];
            const float v[3] = {lo.x + hi.x, lo.y + hi.y, lo.z + hi.z};
            key = 0;
            for (int k = 0; k < 3; ++k) {
                const float ext = ce[3 + k] - ce[k];
                const float u = ext > 0.0f ? (v[k] - ce[k]) / ext * 64.0f : 0.0f;
                const uint32_t q = (uint32_t)fminf(fmaxf(u, 0.0f), 63.0f);
                for (int b = 0; b < 6; ++b) key |= (q >> b & 1u) << (3 * b + 2 - k);
            }
            key = key << 13 | (uint32_t)s;
        }
        keys[s] = key;
    }
    for (int size = 2; size <= n2; size <<= 1)
        for (int st = size >> 1; st > 0; st >>= 1) {
            top_barrier();
            for (int i = tid; i < n2 / 2; i += T) {
                const int a = 2 * i - (i & (st - 1)), b = a + st;
                const uint32_t x = keys[a], y = keys[b];
                if ((x > y) == ((a & size) == 0)) {
                    keys[a] = y;
                    keys[b] = x;
                }
            }
        }
    top_barrier();
    for (int i = tid; i < n; i += T) order_out[i] = (int32_t)(keys[i] & 8191u);
    for (int g = wave; g < n_group; g += NW) {
        const int a = top_group(g, n_group, n), b = top_group(g + 1, n_group, n);
        float m[6] = {3e38f, 3e38f, 3e38f, -3e38f, -3e38f, -3e38f}, w = 0.0f;
        for (int i = a + lane; i < b; i += 64) {
            const int s = (int)(keys[i] & 8191u);
            const float4 lo = sb[2 * s], hi = sb[2 * s + 1];
            const float v[6] = {lo.x, lo.y, lo.z, hi.x, hi.y, hi.z};
            for (int k = 0; k < 3; ++k) {
                m[k] = fminf(m[k], v[k]);
                m[3 + k] = fmaxf(m[3 + k], v[3 + k]);
            }
            w += lo.w;
        }
        for (int k = 0; k < 3; ++k) {
            m[k] = -wave_max(-m[k]);
            m[3 + k] = wave_max(m[3 + k]);
        }
        for (int d = 32; d > 0; d >>= 1) w += __shfl_xor(w, d, 64);
        if (lane == 0) {
            sh.box[2 * g] = make_float4(m[0], m[1], m[2], w);
            sh.box[2 * g + 1] = make_float4(m[3], m[4], m[5], 0.0f);
            sh.ids[g] = ids[b - 1];   // a group's own nodes take those of a .. b - 2
        }
    }
    top_barrier();
    for (int g = tid; g < n_group; g += T) sh.idx[g] = (uint16_t)g;
}

// Upper levels, one workgroup: the surfaces' subtree boxes into sb, ranges
// split until they hold at most TOP_LEAF surfaces; those go to fin (start, end,
// parent, side) and the surfaces' order to order_out.  Or, grouped: the groups
// split to the end, each of them to fin.
__global__ __launch_bounds__(TOP_T) void k_top_split(const int32_t* s_ptr, const int32_t* n_surf_p,
                                                     const int32_t* seen_p, int64_t n_tri, const int2* range,
                                                     const float* lbox, float4* sb, int32_t* ids, int32_t* order_out,
                                                     int4* fin, int32_t* n_fin, TopOut o)
{
    __shared__ TopShared<RT_TOP_MAX, TOP_RES, TOP_T, TOP_Q> sh;
    const int n = *n_surf_p;
    if (!top_used(n, *seen_p)) return;   // the same for every thread
    const bool grouped = !top_full(n, n_tri), resident = !grouped && n <= TOP_RES;
    const int leaf = grouped || n <= TOP_LEAF ? 1 : TOP_LEAF;
    float ce[6] = {3e38f, 3e38f, 3e38f, -3e38f, -3e38f, -3e38f};   // extent of the doubled centres
    for (int s = threadIdx.x; s < n; s += TOP_T) {
        // the surface's leaves are slots a..b-1; its subtree's node has index a or b - 1
        const int a = s_ptr[s], b = s_ptr[s + 1];
        float4 lo, hi;
        int ref, free = a;
        if (b - a == 1) {
            ref = ~a;
            const float* x = lbox + 6 * (int64_t)a;
            lo = make_float4(x[0], x[1], x[2], 1.0f);
            hi = make_float4(x[3], x[4], x[5], 0.0f);
        } else {
            const int2 ra = range[a];
            ref = ra.x == a && ra.y == b - 1 ? a : b - 1;
            free = ref == a ? b - 1 : a;
            const float4* nd = o.nodes + 4 * (int64_t)ref;
            const float4 l0 = nd[0], l1 = nd[1], r0 = nd[2], r1 = nd[3];
            lo = make_float4(fminf(l0.x, r0.x), fminf(l0.y, r0.y), fminf(l0.z, r0.z), (float)(b - a));
            hi = make_float4(fmaxf(l1.x, r1.x), fmaxf(l1.y, r1.y), fmaxf(l1.z, r1.z), 0.0f);
        }
        hi.w = __int_as_float(ref);
        if (grouped || leaf > 1) {
            sb[2 * s] = lo;
            sb[2 * s + 1] = hi;
            ids[s] = free;
        }
        if (resident) {
            sh.ids[s] = free;
            sh.box[2 * s] = lo;
            sh.box[2 * s + 1] = hi;
        }
        if (grouped) {
            const float v[3] = {lo.x + hi.x, lo.y + hi.y, lo.z + hi.z};
            for (int k = 0; k < 3; ++k) {
                ce[k] = fminf(ce[k], v[k]);
                ce[3 + k] = fmaxf(ce[3 + k], v[k]);
            }
        } else {
            sh.idx[s] = (uint16_t)s;
        }
    }
    const int n_group = grouped ? (n + TOP_GROUP - 1) / TOP_GROUP : 0;
    if (grouped) top_groups(sh, n, n_group, ce, sb, ids, order_out);
    const int n_item = grouped ? n_group : n;
    if (threadIdx.x == 0) {
        sh.nq[0] = 1;
        sh.nq[1] = 0;
        sh.nfin = 0;
        sh.queue[0][0] = make_int4(0, n_item, -1, 0);
    }
    __syncthreads();
    o.ids = grouped || resident ? sh.ids : ids;
    if (grouped || resident)
        top_levels(sh, TopBoxes{sh.box}, n_item, leaf, n_group, n, fin, o);
    else
        top_levels(sh, TopBoxes{sb}, n_item, leaf, 0, n, fin, o);
    if (leaf > 1)
        for (int i = threadIdx.x; i < n; i += TOP_T) order_out[i] = sh.idx[i];
    if (threadIdx.x == 0) *n_fin = sh.nfin;
}

// Lower levels: one workgroup per range of at most TOP_LEAF surfaces, split to the end.
__global__ __launch_bounds__(TOP_FT) void k_top_finish(const int32_t* n_surf_p, const int32_t* seen_p,
                                                       const float4* sb, const int32_t* ids, const int32_t* order,
                                                       const int4* fin, const int32_t* n_fin, TopOut o)
{
    __shared__ TopShared<TOP_LEAF, TOP_LEAF, TOP_FT, TOP_Q> sh;
    if (!top_used(*n_surf_p, *seen_p) || (int)blockIdx.x >= *n_fin) return;   // the same for every thread
    const int4 root = fin[blockIdx.x];
    const int a0 = root.x, cnt = root.y - a0;
    if ((int)threadIdx.x < cnt) {
        const int s = order[a0 + threadIdx.x];
        sh.idx[threadIdx.x] = (uint16_t)threadIdx.x;
        sh.ids[threadIdx.x] = ids[a0 + threadIdx.x];   // positions within the range
        sh.box[2 * threadIdx.x] = sb[2 * s];
        sh.box[2 * threadIdx.x + 1] = sb[2 * s + 1];
    }
    if (threadIdx.x == 0) {
        sh.nq[0] = 1;
        sh.nq[1] = 0;
        sh.queue[0][0] = make_int4(0, cnt, root.z, root.w);
    }
    __syncthreads();
    o.ids = sh.ids;
    top_levels(sh, TopBoxes{sh.box}, cnt, 1, 0, cnt, nullptr, o);
}

// 4-wide nodes: every internal node of even depth lists its
// grandchildren (a leaf child stands for itself).  Boxes are copied from the
// binary nodes.  Also the tree depth: the deepest leaf lies one below the
// deepest internal node (a broken parent chain gives 2^20).
// blockIdx.y 1: the Morton tree's depth, and its leaf links turned into slots.
struct MortonTree {
    const uint64_t* keys;
    const int32_t* parent_int;
    const int32_t* tslot;      // slot of each triangle
    int32_t* child;
    int32_t* maxd;
};
__global__ void k_node4(const int32_t* child, const int32_t* parent_int, const float4* nodes, const float4* tri4,
                        int64_t ni, float4* node4, int32_t* maxd, MortonTree mt)
{
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool second = blockIdx.y != 0;
    const int32_t* up = second ? mt.parent_int : parent_int;
    const bool live = n < ni;
    int d = 0;
    int32_t p = live ? up[n] : -1;
    for (; p >= 0 && p < ni && d < 4096; p = up[p]) ++d;
    const unsigned dl = !live ? 0u : (p != -1 ? (1u << 20) : (unsigned)d + 1u);
    const unsigned dm = wave_umax(dl);
    if ((threadIdx.x & 63) == 0 && dm > 0) atomicMax(second ? mt.maxd : maxd, (int32_t)dm);
    if (second) {
        if (live)
            for (int side = 0; side < 2; ++side) {
                const int32_t c = mt.child[2 * n + side];
                if (c < 0) mt.child[2 * n + side] = ~mt.tslot[mt.keys[2 * (int64_t)(~c)]];
            }
        return;
    }
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
// 119 us for 1566 surfaces of 128 triangles; 27 us so, 14 of them for the lists
// of a grid finer than 4 x 4).
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
// overlaps.  Lists keep the surface's triangle order.  At least as many cells
// as triangles (2 x 2 to 32 x 32), halved per axis until the lists fit their
// part of g_tris: with 4 x 4 cells for every surface, a point on an office's
// floor tile of 800 triangles met some 36 of them one behind the other, 19 of
// the 46 ms of its per-element kernel (31 ms so; geometry of the two sources
// 5.6 and 4.6 ms, 2.3 and 1.6 so).
//
// The lists of 64 triangles at a time: their bits in the cells' masks in LDS
// (any order), then every cell's lane appends its bits' triangles in order.
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

__global__ __launch_bounds__(256) void k_surf_tables(const int32_t* s_ptr, const int32_t* s_tris, const float* verts,
                                                     const double* t_edge, const int32_t* n_surf_p, double* s_plane, double* s_box,
                                                     int32_t* g_axes, double* g_frame, int32_t* g_off,
                                                     int32_t* g_tris, int32_t* bad)
{
    constexpr int CELLS = 1 << (2 * RT_SGRID_HI);
    __shared__ int l_cnt[4][CELLS];                  // per wave and cell: triangles listed so far
    __shared__ unsigned long long l_mask[4][CELLS];  // and those of the 64 at hand
    const int lane = threadIdx.x & 63;
    volatile int* cnt = l_cnt[threadIdx.x >> 6];
    volatile unsigned long long* mask = l_mask[threadIdx.x >> 6];
    const int n_surf = *n_surf_p;
    for (int s = (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)); s < n_surf;
         s += (int)(gridDim.x * (blockDim.x >> 6))) {
        const int b = s_ptr[s], e = s_ptr[s + 1];
        if (b >= e) {   // an unused id (reported as invalid)
            if (lane < RT_PLANE) s_plane[RT_PLANE * (int64_t)s + lane] = 0.0;
            if (lane < 6) s_box[6 * (int64_t)s + lane] = lane < 3 ? 1e300 : -1e300;
            if (lane == 0) g_axes[s] = -1;
            continue;
        }
        const float* first = verts + 9 * (int64_t)s_tris[b];
        double v[3], e1[3], e2[3];
        for (int k = 0; k < 3; ++k) {
            v[k] = first[k];
            e1[k] = (double)first[3 + k] - v[k];
            e2[k] = (double)first[6 + k] - v[k];
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
            const float* p = verts + 9 * (int64_t)t;
            for (int a = 0; a < 3; ++a) {
                const double w[3] = {p[3 * a], p[3 * a + 1], p[3 * a + 2]};
                for (int k = 0; k < 3; ++k) {
                    lo[k] = fmin(lo[k], w[k]);
                    hi[k] = fmax(hi[k], w[k]);
                }
                const double dist = n0 * w[0] + n1 * w[1] + n2 * w[2] - dpl;
                off_plane |= !(fabs(dist) <= tol);
            }
            const int ax = edge_axes(t_edge, t);
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
            double* pl = s_plane + RT_PLANE * (int64_t)s;
            const double nn = n0 * n0 + n1 * n1 + n2 * n2;
            pl[0] = n0;
            pl[1] = n1;
            pl[2] = n2;
            pl[3] = dpl;
            pl[4] = nn;
            pl[5] = 1.0 / nn;
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
        if (!grid) {
            if (lane == 0) g_axes[s] = -1;
            continue;
        }
        const int n = e - b;
        int lg = RT_SGRID_LO;
        while (lg < RT_SGRID_HI && (1 << (2 * lg)) < n) ++lg;
        double pu, pv;
        // cells of triangle j of the surface, first and last along u and v, a byte each; t: the triangle, -1: none
        auto cells_of = [&](int j, int& t) {
            t = -1;
            if (j >= e) return 0u;
            const int tj = s_tris[j];
            if (edge_axes(t_edge, tj) & 16) return 0u;   // a degenerate triangle contains nothing
            t = tj;
            const float* p = verts + 9 * (int64_t)t;
            const double q[6] = {p[i0], p[i1], p[3 + i0], p[3 + i1], p[6 + i0], p[6 + i1]};
            const double umin = fmin(q[0], fmin(q[2], q[4])), umax = fmax(q[0], fmax(q[2], q[4]));
            const double vmin = fmin(q[1], fmin(q[3], q[5])), vmax = fmax(q[1], fmax(q[3], q[5]));
            const double C = fmax(fmax(fabs(umin), fabs(umax)), fmax(fabs(vmin), fabs(vmax)));
            auto sq = [](double x, double y) { return x * x + y * y; };
            const double l2 = fmin(sq(q[2] - q[0], q[3] - q[1]),
                                   fmin(sq(q[4] - q[2], q[5] - q[3]), sq(q[0] - q[4], q[1] - q[5])));
            const double lmin = fmax(sqrt(l2), 1e-300);
            const double m = 1e-13 * (C * C / lmin) + 1e-9 * C + 1e-12;
            const unsigned c0 = sgrid_index(umin - m, u0, pu, lg), c1 = sgrid_index(umax + m, u0, pu, lg);
            const unsigned d0 = sgrid_index(vmin - m, v0, pv, lg), d1 = sgrid_index(vmax + m, v0, pv, lg);
            return c0 | c1 << 8 | d0 << 16 | d1 << 24;
        };
        auto each_cell = [&](unsigned r, auto f) {
            for (unsigned i = r & 255u; i <= (r >> 8 & 255u); ++i)
                for (unsigned k = r >> 16 & 255u; k <= r >> 24; ++k) f((i << lg) + k);
        };
        // between phases that hand LDS words from lane to lane (one wave: its LDS operations keep their order)
        auto handed = [] {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        int t, first_t[2] = {-1, -1};             // the first 128 triangles stay in registers
        unsigned cells, first_cells[2] = {0, 0};
        for (;; --lg) {
            pu = eu > 0.0 ? (double)(1 << lg) / eu : 0.0;
            pv = ev > 0.0 ? (double)(1 << lg) / ev : 0.0;
            for (int c = lane; c < 1 << (2 * lg); c += 64) {
                cnt[c] = 0;
                mask[c] = 0ull;
            }
            handed();
            long long total = 0;
            for (int j0 = b; j0 < e; j0 += 64) {
                cells = cells_of(j0 + lane, t);
                if (j0 == b) first_t[0] = t, first_cells[0] = cells;
                if (j0 == b + 64) first_t[1] = t, first_cells[1] = cells;
                if (t < 0) continue;
                total += (int)(((cells >> 8 & 255u) - (cells & 255u) + 1u) * ((cells >> 24) - (cells >> 16 & 255u) + 1u));
                each_cell(cells, [&](unsigned c) { atomicAdd((int*)&cnt[c], 1); });
            }
            handed();
            for (int o = 32; o > 0; o >>= 1) total += __shfl_xor(total, o, 64);
            if (lg == RT_SGRID_LO || total <= (long long)RT_SGRID_CAP * n) break;
        }
        const int nc = 1 << (2 * lg);
        if (lane == 0) {
            g_axes[s] = amax | lg << 4;
            double* f = g_frame + 4 * (int64_t)s;
            f[0] = u0;
            f[1] = v0;
            f[2] = pu;
            f[3] = pv;
        }
        // counts to first places
        int32_t* off = g_off + (int64_t)RT_SGRID_OFF * b + s;
        int32_t* list = g_tris + (int64_t)RT_SGRID_CAP * b;
        int run = 0;
        for (int c = lane; c < ((nc + 63) & ~63); c += 64) {   // every lane the same number of times
            const int v = c < nc ? cnt[c] : 0;
            int x = v;
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(x, o, 64);
                if (lane >= o) x += y;
            }
            if (c < nc) {
                off[c] = run + x - v;
                cnt[c] = run + x - v;
            }
            run += __shfl(x, 63, 64);
        }
        if (lane == 0) off[nc] = run;
        for (int j0 = b; j0 < e; j0 += 64) {
            if (j0 < b + 128) {
                t = j0 == b ? first_t[0] : first_t[1];
                cells = j0 == b ? first_cells[0] : first_cells[1];
            } else {
                cells = cells_of(j0 + lane, t);
            }
            if (t >= 0)
                each_cell(cells, [&](unsigned c) { atomicOr((unsigned long long*)&mask[c], 1ull << lane); });
            handed();
            for (int c = lane; c < ((nc + 63) & ~63); c += 64) {
                unsigned long long m = c < nc ? mask[c] : 0ull;
                int at = c < nc ? cnt[c] : 0;
                if (m) mask[c] = 0ull;
                while (__ballot(m != 0ull) != 0ull) {
                    const int from = m ? __builtin_ctzll(m) : 0;
                    const int tt = __shfl(t, from, 64);
                    if (m) list[at++] = tt;
                    m &= m - 1ull;
                }
                if (c < nc) cnt[c] = at;
            }
            handed();
        }
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
__global__ void k_unit_normals(const float* verts, int64_t nt, double* nrm)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nt) return;
    double v[9];
    for (int k = 0; k < 9; ++k) v[k] = verts[9 * t + k];
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
    hipLaunchKernelGGL(k_unit_normals, dim3(blocks_for(s.n_tri, 256)), dim3(256), 0, st, s.verts.as<float>(), s.n_tri,
                       s.nrm.as<double>());
    HIP_CHECK(hipGetLastError());
}

// Boxes of the scene's Morton tree for a counting walk (nodes as SceneView
// lays them out, root 0), made on `st` when one is asked for: leaf boxes from
// the nodes that hold them, then the leaf-to-root walk with device-wide
// arrival counts (fences at every level: slow, and only taken here).
__global__ void k_leaf_boxes(const float4* nodes, int64_t n_nodes, int64_t nt, float* lbox)
{
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= n_nodes) return;
    for (int side = 0; side < 2; ++side) {
        const int32_t ref = ((const int32_t*)nodes)[16 * n + 4 * side + 3];
        if (ref >= 0 || ~ref >= nt) continue;
        const float4 l = nodes[4 * n + 2 * side], h = nodes[4 * n + 2 * side + 1];
        float* b = lbox + 6 * (int64_t)(~ref);
        b[0] = l.x;
        b[1] = l.y;
        b[2] = l.z;
        b[3] = h.x;
        b[4] = h.y;
        b[5] = h.z;
    }
}

__global__ void k_parents(const int32_t* child, int64_t ni, int32_t* parent_int, int32_t* parent_leaf)
{
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= ni) return;
    if (n == 0) parent_int[0] = -1;
    for (int side = 0; side < 2; ++side) {
        const int32_t c = child[2 * n + side];
        if (c < 0)
            parent_leaf[~c] = (int32_t)n;
        else
            parent_int[c] = (int32_t)n;
    }
}

__device__ __forceinline__ void load_box(int32_t c, const float* lbox, const float* ibox, float* b)
{
    const volatile float* src = c < 0 ? (const volatile float*)(lbox + 6 * (int64_t)(~c))
                                      : (const volatile float*)(ibox + 6 * (int64_t)c);
    for (int k = 0; k < 6; ++k) b[k] = src[k];
}

__global__ void k_refit(const int32_t* child, const int32_t* parent_int, const int32_t* parent_leaf,
                        const float* lbox, float* ibox, int32_t* flags, float4* nodes, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int32_t p = parent_leaf[i];
    while (p >= 0 && p < n - 1) {
        __threadfence();
        int old = __hip_atomic_fetch_add(&flags[p], 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (old == 0) return;
        int32_t cl = child[2 * p], cr = child[2 * p + 1];
        float bl[6], br[6];
        load_box(cl, lbox, ibox, bl);
        load_box(cr, lbox, ibox, br);
        nodes[4 * (int64_t)p + 0] = make_float4(bl[0], bl[1], bl[2], __int_as_float(cl));
        nodes[4 * (int64_t)p + 1] = make_float4(bl[3], bl[4], bl[5], __int_as_float(cr));
        nodes[4 * (int64_t)p + 2] = make_float4(br[0], br[1], br[2], 0.0f);
        nodes[4 * (int64_t)p + 3] = make_float4(br[3], br[4], br[5], 0.0f);
        volatile float* dst = ibox + 6 * (int64_t)p;
        for (int k = 0; k < 3; ++k) {
            dst[k] = fminf(bl[k], br[k]);
            dst[3 + k] = fmaxf(bl[3 + k], br[3 + k]);
        }
        __threadfence();
        p = parent_int[p];
    }
}

__global__ void k_zero_i32(int32_t* p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

void lbvh_nodes(Ctx& c, const Scene& s, Scratch& nodes, hipStream_t st)
{
    const int64_t nt = s.n_tri, ni = nt - 1;
    if (ni <= 0) return;
    const int B = 256;
    nodes = Scratch(c, sizeof(float4) * 4 * (size_t)ni, st);
    Scratch lbox(c, sizeof(float) * 6 * (size_t)nt, st), ibox(c, sizeof(float) * 6 * (size_t)ni, st),
        pint(c, sizeof(int32_t) * (size_t)ni, st), pleaf(c, sizeof(int32_t) * (size_t)nt, st),
        flags(c, sizeof(int32_t) * (size_t)ni, st);
    hipLaunchKernelGGL(k_zero_i32, dim3(blocks_for(ni, B)), dim3(B), 0, st, flags.as<int32_t>(), ni);
    HIP_CHECK(hipGetLastError());
    hipLaunchKernelGGL(k_leaf_boxes, dim3(blocks_for(ni, B)), dim3(B), 0, st, s.nodes.as<float4>(), ni, nt,
                       lbox.as<float>());
    HIP_CHECK(hipGetLastError());
    hipLaunchKernelGGL(k_parents, dim3(blocks_for(ni, B)), dim3(B), 0, st, s.lbvh_child.as<int32_t>(), ni,
                       pint.as<int32_t>(), pleaf.as<int32_t>());
    HIP_CHECK(hipGetLastError());
    hipLaunchKernelGGL(k_refit, dim3(blocks_for(nt, B)), dim3(B), 0, st, s.lbvh_child.as<int32_t>(),
                       pint.as<int32_t>(), pleaf.as<int32_t>(), lbox.as<float>(), ibox.as<float>(),
                       flags.as<int32_t>(), nodes.as<float4>(), nt);
    HIP_CHECK(hipGetLastError());
}

// plain: no tree above the surfaces (one linear BVH over the whole scene)
static void build_scene_as(Ctx& c, Scene& s, const float* V, int64_t nv, const int32_t* T, int64_t nt,
                           const int32_t* surf, const float* rr, const float* ri, bool plain, hipStream_t st)
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

    s.verts = Scratch(c, sizeof(float) * 9 * (size_t)nt, st);
    s.t_edge = Scratch(c, sizeof(double) * RT_EDGE * (size_t)nt, st);
    s.refl = Scratch(c, sizeof(float2) * (size_t)nt, st);
    s.surf = Scratch(c, sizeof(int32_t) * (size_t)nt, st);
    s.tri4 = Scratch(c, sizeof(float4) * 3 * (size_t)nt, st);
    Scratch cent(c, sizeof(float4) * (size_t)nt, st);
    // control block: bounds[12] unsigned, bad, depth of the Morton tree, n_surf, seen, nodes spanning several
    // refit tiles, depth of the walked tree, its root, ranges left by k_top_split
    Scratch ctl(c, 64 * sizeof(int32_t), st);
    unsigned* bounds = ctl.as<unsigned>();
    int32_t* bad = ctl.as<int32_t>() + 12;
    int32_t* maxd = ctl.as<int32_t>() + 13;
    int32_t* nsurf = ctl.as<int32_t>() + 14;
    int32_t* seen = ctl.as<int32_t>() + 15;
    int32_t* ncross = ctl.as<int32_t>() + 16;
    int32_t* wmaxd = ctl.as<int32_t>() + 17;
    int32_t* troot = ctl.as<int32_t>() + 18;
    int32_t* nfin = ctl.as<int32_t>() + 19;
    hipLaunchKernelGGL(k_ctl_init, dim3(1), dim3(64), 0, st, bounds);
    HIP_CHECK(hipGetLastError());
    const int B = 256;
    Scratch skeys(c, sizeof(uint64_t) * (size_t)nt, st);
    hipLaunchKernelGGL(k_scene_prep, dim3(std::min<unsigned>(blocks_for(nt, PREP_B), PREP_BLOCKS)), dim3(PREP_B), 0, st,
                       dV, dT, dS, dR, dI, nv, nt, s.verts.as<float>(), s.refl.as<float2>(), s.surf.as<int32_t>(),
                       cent.as<float4>(), skeys.as<uint64_t>(), bounds, bad, nsurf, s.t_edge.as<double>());
    HIP_CHECK(hipGetLastError());
    s.box = Scratch(c, 6 * sizeof(float), st);
    Scratch keys_raw(c, 2 * sizeof(uint64_t) * (size_t)nt, st), keys(c, 2 * sizeof(uint64_t) * (size_t)nt, st);
    hipLaunchKernelGGL(k_morton, dim3(blocks_for(nt, B)), dim3(B), 0, st, cent.as<float4>(), bounds, nt,
                       keys_raw.as<uint64_t>(), s.box.as<float>());
    HIP_CHECK(hipGetLastError());
    sort_keys(c, keys_raw.as<uint64_t>(), keys.as<uint64_t>(), nt, 2, 64, 127, st);
    // surfaces (tables sized for the largest valid count, n_surf <= n_tri)
    int sbits = 1;
    while (((int64_t)1 << sbits) < nt) ++sbits;
    {
        // the keys come in triangle order and the sort is stable: the surface bits decide alone
        Scratch sorted(c, sizeof(uint64_t) * (size_t)nt, st);
        sort_keys(c, skeys.as<uint64_t>(), sorted.as<uint64_t>(), nt, 1, 32, 32 + sbits, st);
        std::swap(skeys, sorted);
    }
    s.s_ptr = Scratch(c, sizeof(int32_t) * (size_t)(nt + 1), st);
    s.s_tris = Scratch(c, sizeof(int32_t) * (size_t)nt, st);
    s.s_plane = Scratch(c, sizeof(double) * RT_PLANE * (size_t)nt, st);
    s.s_box = Scratch(c, sizeof(double) * 6 * (size_t)nt, st);
    hipLaunchKernelGGL(k_surf_csr, dim3(blocks_for(nt, B)), dim3(B), 0, st, skeys.as<uint64_t>(), nt, nsurf,
                       s.s_ptr.as<int32_t>(), s.s_tris.as<int32_t>(), seen);
    HIP_CHECK(hipGetLastError());
    // leaf slots: by surface, then Morton code
    Scratch slots(c, 2 * sizeof(uint64_t) * (size_t)nt, st), tslot(c, sizeof(int32_t) * (size_t)nt, st);
    hipLaunchKernelGGL(k_slot_keys, dim3(blocks_for(nt, B)), dim3(B), 0, st, keys.as<uint64_t>(), s.surf.as<int32_t>(),
                       nt, nsurf, plain ? 1 : 0, keys_raw.as<uint64_t>());
    HIP_CHECK(hipGetLastError());
    int tbits = 0;   // surfaces take part up to RT_TOP_MAX of them
    while (tbits < sbits && (1 << tbits) < RT_TOP_MAX) ++tbits;
    sort_keys(c, keys_raw.as<uint64_t>(), slots.as<uint64_t>(), nt, 2, 64 + RT_KEY_SURF_SHIFT,
              64 + RT_KEY_SURF_SHIFT + tbits, st);
    Scratch lbox(c, sizeof(float) * 6 * (size_t)nt, st);
    hipLaunchKernelGGL(k_leaves, dim3(blocks_for(nt, B)), dim3(B), 0, st, slots.as<uint64_t>(), dV, dT,
                       s.surf.as<int32_t>(), nv, nt, bounds, s.tri4.as<float4>(), lbox.as<float>(),
                       tslot.as<int32_t>());
    HIP_CHECK(hipGetLastError());

    if (nt >= 2) {
        const int64_t ni = nt - 1;
        s.nodes = Scratch(c, sizeof(float4) * 4 * (size_t)ni, st);
        s.lbvh_child = Scratch(c, sizeof(int32_t) * 2 * (size_t)ni, st);
        const int64_t n_tiles = (nt + RT_REFIT_TILE - 1) / RT_REFIT_TILE;
        Scratch child(c, sizeof(int32_t) * 2 * (size_t)ni, st), pint(c, sizeof(int32_t) * (size_t)ni, st),
            pleaf(c, sizeof(int32_t) * (size_t)nt, st), range(c, sizeof(int2) * (size_t)ni, st),
            cross(c, sizeof(int32_t) * (size_t)(n_tiles > 1 ? ni : 1), st),
            tbox(c, sizeof(float) * 6 * (size_t)n_tiles, st), mpint(c, sizeof(int32_t) * (size_t)ni, st);
        const KarrasOut ko{slots.as<uint64_t>(), child.as<int32_t>(), pint.as<int32_t>(), pleaf.as<int32_t>()};
        const KarrasOut km{keys.as<uint64_t>(), s.lbvh_child.as<int32_t>(), mpint.as<int32_t>(), nullptr};
        hipLaunchKernelGGL(k_karras, dim3(blocks_for(ni, B), 2), dim3(B), 0, st, ko, km, nt, range.as<int2>(),
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
        if (!plain) {
            const int64_t ns = std::min<int64_t>(nt, RT_TOP_MAX);
            Scratch sb(c, sizeof(float4) * 2 * (size_t)ns, st), ids(c, sizeof(int32_t) * (size_t)ns, st),
                order(c, sizeof(int32_t) * (size_t)ns, st), fin(c, sizeof(int4) * (size_t)ns, st);
            const TopOut to{s.nodes.as<float4>(), child.as<int32_t>(), pint.as<int32_t>(), troot, nullptr};
            hipLaunchKernelGGL(k_top_split, dim3(1), dim3(TOP_T), 0, st, s.s_ptr.as<int32_t>(), nsurf, seen, nt,
                               range.as<int2>(), lbox.as<float>(), sb.as<float4>(), ids.as<int32_t>(),
                               order.as<int32_t>(), fin.as<int4>(), nfin, to);
            HIP_CHECK(hipGetLastError());
            hipLaunchKernelGGL(k_top_finish, dim3((unsigned)std::max<int64_t>(1, ns / 2)), dim3(TOP_FT), 0, st, nsurf, seen,
                               sb.as<float4>(), ids.as<int32_t>(), order.as<int32_t>(), fin.as<int4>(), nfin, to);
            HIP_CHECK(hipGetLastError());
        }
        s.node4 = Scratch(c, sizeof(float4) * 8 * (size_t)ni, st);
        const MortonTree mt{keys.as<uint64_t>(), mpint.as<int32_t>(), tslot.as<int32_t>(), s.lbvh_child.as<int32_t>(),
                            maxd};
        hipLaunchKernelGGL(k_node4, dim3(blocks_for(ni, B), 2), dim3(B), 0, st, child.as<int32_t>(),
                           pint.as<int32_t>(), s.nodes.as<float4>(), s.tri4.as<float4>(), ni,
                           s.node4.as<float4>(), wmaxd, mt);
        HIP_CHECK(hipGetLastError());
    }
    // the tree's scratch goes back before the tables below are allocated
    for (Scratch* p : {&cent, &keys_raw, &keys, &skeys, &slots, &tslot, &lbox}) p->release();

    s.g_axes = Scratch(c, sizeof(int32_t) * (size_t)nt, st);
    s.g_frame = Scratch(c, sizeof(double) * 4 * (size_t)nt, st);
    s.g_off = Scratch(c, sizeof(int32_t) * (RT_SGRID_OFF + 1) * (size_t)nt, st);   // n_surf <= nt
    s.g_tris = Scratch(c, sizeof(int32_t) * RT_SGRID_CAP * (size_t)nt, st);
    hipLaunchKernelGGL(k_surf_tables, dim3(std::min<unsigned>(blocks_for(nt, 4), 2048)), dim3(256), 0, st,
                       s.s_ptr.as<int32_t>(), s.s_tris.as<int32_t>(), s.verts.as<float>(), s.t_edge.as<double>(),
                       nsurf, s.s_plane.as<double>(), s.s_box.as<double>(),
                       s.g_axes.as<int32_t>(), s.g_frame.as<double>(), s.g_off.as<int32_t>(),
                       s.g_tris.as<int32_t>(), bad);
    HIP_CHECK(hipGetLastError());
    // one read-back: input checks, tree checks, surface count
    int64_t hq[4];
    read_i64s((const int64_t*)(ctl.as<int32_t>() + 12), hq, 4, st);
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
    const int32_t wdepth = (int32_t)(hq[2] >> 32);
    const bool top = !plain && top_wanted(n_surf);
    s.walk_depth = wdepth;
    s.root = nt < 2 ? ~0 : top ? (int32_t)(hq[3] & 0xffffffff) : 0;
    if (top && (s.root < 0 || s.root >= nt - 1 || wdepth >= (1 << 20)))
        throw hip_error("BVH build produced an inconsistent tree");
}

void build_scene(Ctx& c, Scene& s, const float* V, int64_t nv, const int32_t* T, int64_t nt,
                 const int32_t* surf, const float* rr, const float* ri, hipStream_t st)
{
    build_scene_as(c, s, V, nv, T, nt, surf, rr, ri, false, st);
    // deeper than the stacks hold (chains of surfaces nested in one another): the linear BVH, whose depth was checked
    if (s.walk_depth > RT_STACK - 1) build_scene_as(c, s, V, nv, T, nt, surf, rr, ri, true, st);
}

}  // namespace rt
