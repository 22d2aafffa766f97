// Internal declarations of the risrt library (gfx950).
//
// Geometry decisions follow fixed formulas so that results are reproducible:
//   * ray/triangle: Moller-Trumbore in FP32, left-to-right sums, no fused
//     multiply-add, one correctly rounded division (1 / det);
//   * specular bounce: d' = d - (2 (d.n) / (n.n)) n, n = e1 x e2, FP32;
//   * image method, containment, side tests, lengths and phase: FP64 without
//     fused multiply-add.
// Files that include this header compile with contraction off.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <stdexcept>
#include <string>

#include "rt_fp64_core.hpp"
#include "rt_rules.hpp"

#define RT_MAX_K 5            // largest reflection order (keys of two 64-bit words above 3)
#define RT_KM_SMALL 3        // orders up to this use one-word keys and the smaller kernel instances
#define RT_STACK 64          // BVH traversal stack entries per lane (LDS)
#define RT_EPS 1e-4          // metres: legs and bounces ignore hits closer than this
#define RT_KEY_BITS 21

namespace rt {

struct hip_error : std::runtime_error {
    explicit hip_error(const std::string& s) : std::runtime_error(s) {}
};

#define HIP_CHECK(x)                                                                        \
    do {                                                                                    \
        hipError_t e_ = (x);                                                                \
        if (e_ != hipSuccess)                                                               \
            throw ::rt::hip_error(std::string(#x) + ": " + hipGetErrorString(e_));           \
    } while (0)

// --------------------------------------------------------------------------
// Device views
// --------------------------------------------------------------------------
struct SceneView {
    int32_t n_tri;
    int32_t n_surf;
    int32_t root;          // >= 0 internal node, < 0 leaf ~slot; unused if n_tri == 0
    int32_t pad;
    const float4* tri4;    // 3 per leaf slot: (v0, id), (e1, surf), (e2, 0)
    const float4* nodes;   // 4 per internal node: (loL, cL), (hiL, cR), (loR, -), (hiR, -)
    const float4* node4;   // 8 per internal node of even depth (4-wide collapse), see RT_NODE4
    const float2* refl;    // per triangle
    const float2* mat;     // per triangle: relative permittivity, conductivity S/m (null: none set)
    const double* nrm;     // per triangle unit normal e1 x e2 / |e1 x e2| (FP64), set with the materials
    const int32_t* surf;   // per triangle
    const int32_t* s_ptr;  // n_surf + 1
    const int32_t* s_tris; // triangles grouped by surface, ascending
    const double* s_plane; // RT_PLANE per surface: n (not unit), c = n . v0 of its first triangle, n . n, 1 / (n . n)
    const double* s_box;   // 6 per surface: lo, hi (inflated by 1e-9 m)
    const double* t_edge;  // RT_EDGE per triangle: the edge functions of the containment test, see triangle_edges
    // containment grid per surface: 2^lg x 2^lg cells (lg of RT_SGRID_LO .. RT_SGRID_HI) over the
    // surface box in the projection all its triangles share
    const int32_t* g_axes;   // per surface: the projection's axes | lg << 4; -1: no grid, scan every triangle
    const double* g_frame;   // 4 per surface: u0, v0, cells per unit along u and v
    const int32_t* g_off;    // cell c of surface sf lists [off[c], off[c + 1]) of the surface's part of g_tris,
                             // off = g_off + RT_SGRID_OFF * s_ptr[sf] + sf
    const int32_t* g_tris;   // surface sf's part: from RT_SGRID_CAP * s_ptr[sf] on
};

#define RT_PLANE 6
#define RT_EDGE 13
#define RT_SGRID_LO 1
#define RT_SGRID_HI 5
#define RT_SGRID_OFF 4    // cells of a surface per triangle, at most (the fewest 4^lg that are as many as its triangles)
#define RT_SGRID_CAP 16   // list entries of a surface per triangle, at most

// Grid cell coordinate of x (monotone in x, clamped to the 2^lg cells)
__host__ __device__ __forceinline__ int sgrid_index(double x, double origin, double per_unit, int lg)
{
    double y = (x - origin) * per_unit;
    y = fmin(fmax(y, 0.0), (double)((1 << lg) - 1));
    return (int)y;
}

struct Antenna {
    double axis[3];
    double axis_norm;      // |axis| in FP64
    double gain;
    int32_t pattern;
    double param;
};

struct TraceConst {
    double lambda;
    double two_eta0_pt_gt;   // 2 eta0 P_t G_t
    double tx[3];
    Antenna txa;
    Antenna rxa;
    int32_t K;
    int32_t flags;
    int32_t fresnel;       // 0: fixed coefficients; 1 TE, 2 TM Fresnel coefficients of the materials
    int32_t pad;
    double sig_scale;      // 1 / (omega eps0): eps = eps_r - j sigma sig_scale
    double inv_lambda;     // 1 / lambda (phase in turns = length x this)
    float lam_4pi;         // lambda / (4 pi) in FP32 (free-space amplitude factor over the length)
    int32_t pad2;
};

struct RisView {
    int32_t M;
    int32_t pad;
    const double* elem;    // 3 per element
    const int32_t* order;  // elements in the order the per-element kernel groups them (64 per wave)
    double centre[3];
    double normal[3];      // unit
    double normal_norm;    // |normal| in FP64
    double dy, dz, gain, q;
};

// --------------------------------------------------------------------------
// FP32 ray / triangle (same formula as the definition, no contraction)
// --------------------------------------------------------------------------
__device__ __forceinline__ bool mt_hit(float ox, float oy, float oz, float dx, float dy, float dz,
                                       float4 a, float4 b, float4 c, float tmin, float tmax,
                                       float& t_out)
{
#pragma clang fp contract(off)
    const float e1x = b.x, e1y = b.y, e1z = b.z;
    const float e2x = c.x, e2y = c.y, e2z = c.z;
    float px = dy * e2z - dz * e2y;
    float py = dz * e2x - dx * e2z;
    float pz = dx * e2y - dy * e2x;
    float det = e1x * px + e1y * py + e1z * pz;
    if (det == 0.0f) return false;
    float inv = 1.0f / det;
    float sx = ox - a.x;
    float sy = oy - a.y;
    float sz = oz - a.z;
    float u = (sx * px + sy * py + sz * pz) * inv;
    if (!(u >= 0.0f && u <= 1.0f)) return false;
    float qx = sy * e1z - sz * e1y;
    float qy = sz * e1x - sx * e1z;
    float qz = sx * e1y - sy * e1x;
    float v = (dx * qx + dy * qy + dz * qz) * inv;
    if (!(v >= 0.0f && u + v <= 1.0f)) return false;
    float t = (e2x * qx + e2y * qy + e2z * qz) * inv;
    if (!(t > tmin && t < tmax)) return false;
    t_out = t;
    return true;
}

// May mt_hit accept, by its numerators alone (no division)?  Each bound leaves
// at least 1e-4 relative (the formula's rounding is below 1e-6), and a value
// rejected for its sign is at least 1e-20 of the determinant, far above where
// its quotient could round to zero; so a false answer means mt_hit is false.
__device__ __forceinline__ bool mt_maybe(float ox, float oy, float oz, float dx, float dy, float dz, float4 a,
                                         float4 b, float4 c)
{
#pragma clang fp contract(off)
    const float e1x = b.x, e1y = b.y, e1z = b.z;
    const float e2x = c.x, e2y = c.y, e2z = c.z;
    const float px = dy * e2z - dz * e2y;
    const float py = dz * e2x - dx * e2z;
    const float pz = dx * e2y - dy * e2x;
    const float det = e1x * px + e1y * py + e1z * pz;
    const float sx = ox - a.x;
    const float sy = oy - a.y;
    const float sz = oz - a.z;
    const unsigned sg = __float_as_uint(det) & 0x80000000u;
    const float un = __uint_as_float(__float_as_uint(sx * px + sy * py + sz * pz) ^ sg);   // u |det|
    const float lo = fabsf(det) * -1e-20f, hi = fabsf(det) * 1.0001f;
    const float qx = sy * e1z - sz * e1y;
    const float qy = sz * e1x - sx * e1z;
    const float qz = sx * e1y - sy * e1x;
    const float vn = __uint_as_float(__float_as_uint(dx * qx + dy * qy + dz * qz) ^ sg);   // v |det|
    return !(un < lo || un > hi || vn < lo || un + vn > hi);
}

__device__ __forceinline__ void reflect32(float4 b, float4 c, float& dx, float& dy, float& dz)
{
#pragma clang fp contract(off)
    float nx = b.y * c.z - b.z * c.y;
    float ny = b.z * c.x - b.x * c.z;
    float nz = b.x * c.y - b.y * c.x;
    float dn = dx * nx + dy * ny + dz * nz;
    float nn = nx * nx + ny * ny + nz * nz;
    float k = (2.0f * dn) / nn;
    dx = dx - k * nx;
    dy = dy - k * ny;
    dz = dz - k * nz;
}

// FP64 a / b, and L = sqrt(x) with il = 1 / L, from the hardware's estimates
// (rt_fp64_core.hpp; 8 instead of 11 and 16 instead of 33 instructions).
__device__ __forceinline__ double div_fast(double a, double b) { return div_refine(a, b, __builtin_amdgcn_rcp(b)); }
__device__ __forceinline__ void sqrt_inv(double x, double& L, double& il)
{
    sqrt_refine(x, __builtin_amdgcn_rsq(fmax(x, 1e-300)), &L, &il);
}

// Work counters of the counting build of a kernel (node visits, triangle
// tests, FP64 containment tests).
struct WorkCount {
    uint32_t nodes = 0, tris = 0, contain = 0;
};

// --------------------------------------------------------------------------
// BVH walk.  Boxes are inflated at build time, so the slab test may use FMA:
// it never rejects a box holding a triangle the exact-formula test accepts.
// --------------------------------------------------------------------------
struct RayBox {
    float ix, iy, iz;     // 1 / d (zeros nudged to +-1e-30)
    float oix, oiy, oiz;  // o / d
};

__device__ __forceinline__ RayBox make_raybox(float ox, float oy, float oz, float dx, float dy, float dz)
{
    RayBox r;
    float sx = fabsf(dx) < 1e-30f ? copysignf(1e-30f, dx) : dx;
    float sy = fabsf(dy) < 1e-30f ? copysignf(1e-30f, dy) : dy;
    float sz = fabsf(dz) < 1e-30f ? copysignf(1e-30f, dz) : dz;
    r.ix = 1.0f / sx;
    r.iy = 1.0f / sy;
    r.iz = 1.0f / sz;
    r.oix = ox * r.ix;
    r.oiy = oy * r.iy;
    r.oiz = oz * r.iz;
    return r;
}

__device__ __forceinline__ bool slab(const RayBox& r, float4 lo, float4 hi, float tmin, float tmax,
                                     float& tn)
{
    float t0x = __builtin_fmaf(lo.x, r.ix, -r.oix), t1x = __builtin_fmaf(hi.x, r.ix, -r.oix);
    float t0y = __builtin_fmaf(lo.y, r.iy, -r.oiy), t1y = __builtin_fmaf(hi.y, r.iy, -r.oiy);
    float t0z = __builtin_fmaf(lo.z, r.iz, -r.oiz), t1z = __builtin_fmaf(hi.z, r.iz, -r.oiz);
    float a = fmaxf(fmaxf(fminf(t0x, t1x), fminf(t0y, t1y)), fmaxf(fminf(t0z, t1z), tmin));
    float b = fminf(fminf(fmaxf(t0x, t1x), fmaxf(t0y, t1y)), fminf(fmaxf(t0z, t1z), tmax));
    tn = a;
    return a <= b;
}

// Closest hit: lowest (t, triangle id) among triangles other than skip_tri
// with tmin < t < tmax.  Returns the leaf slot or -1.  `stack` points at this
// lane's column of an LDS array laid out [RT_STACK][stride].
// CNT: count the binary nodes visited and the triangles tested in *wc.
template <bool BRUTE, bool CNT = false>
__device__ int closest_hit(const SceneView& s, float ox, float oy, float oz, float dx, float dy,
                           float dz, float tmin, int skip_tri, int* stack, int stride, float& t_best,
                           int& id_best, WorkCount* wc = nullptr)
{
    t_best = __builtin_inff();
    id_best = 0x7fffffff;
    int slot_best = -1;
    if (s.n_tri == 0) return -1;
    if (BRUTE) {
        for (int i = 0; i < s.n_tri; ++i) {
            float4 a = s.tri4[3 * i], b = s.tri4[3 * i + 1], c = s.tri4[3 * i + 2];
            int id = __float_as_int(a.w);
            if (id == skip_tri) continue;
            float t;
            if (mt_hit(ox, oy, oz, dx, dy, dz, a, b, c, tmin, __builtin_inff(), t)) {
                if (t < t_best || (t == t_best && id < id_best)) {
                    t_best = t;
                    id_best = id;
                    slot_best = i;
                }
            }
        }
        return slot_best;
    }
    RayBox rb = make_raybox(ox, oy, oz, dx, dy, dz);
    int sp = 0;
    int node = s.root;
    while (true) {
        if (node >= 0) {
            if (CNT) wc->nodes++;
            const float4* nd = s.nodes + 4 * node;
            float4 n0 = nd[0], n1 = nd[1], n2 = nd[2], n3 = nd[3];
            float tl, tr;
            bool hl = slab(rb, n0, n1, tmin, t_best, tl);
            bool hr = slab(rb, n2, n3, tmin, t_best, tr);
            int cl = __float_as_int(n0.w), cr = __float_as_int(n1.w);
            if (hl && hr) {
                int nearc = tl <= tr ? cl : cr;
                int farc = tl <= tr ? cr : cl;
                stack[sp * stride] = farc;
                ++sp;
                node = nearc;
                continue;
            } else if (hl) {
                node = cl;
                continue;
            } else if (hr) {
                node = cr;
                continue;
            }
        } else {
            int i = ~node;
            if (CNT) wc->tris++;
            float4 a = s.tri4[3 * i], b = s.tri4[3 * i + 1], c = s.tri4[3 * i + 2];
            int id = __float_as_int(a.w);
            float t;
            if (id != skip_tri && mt_hit(ox, oy, oz, dx, dy, dz, a, b, c, tmin, __builtin_inff(), t)) {
                if (t < t_best || (t == t_best && id < id_best)) {
                    t_best = t;
                    id_best = id;
                    slot_best = i;
                }
            }
        }
        if (sp == 0) break;
        --sp;
        node = stack[sp * stride];
    }
    return slot_best;
}

// Any hit of a triangle not on surface skip_a / skip_b with tmin < t < tmax.
template <bool BRUTE, bool CNT = false>
__device__ bool any_hit(const SceneView& s, float ox, float oy, float oz, float dx, float dy, float dz,
                        float tmin, float tmax, int skip_a, int skip_b, int* stack, int stride,
                        WorkCount* wc = nullptr)
{
    if (s.n_tri == 0) return false;
    if (BRUTE) {
        for (int i = 0; i < s.n_tri; ++i) {
            float4 a = s.tri4[3 * i], b = s.tri4[3 * i + 1], c = s.tri4[3 * i + 2];
            int sf = __float_as_int(b.w);
            if (sf == skip_a || sf == skip_b) continue;
            float t;
            if (CNT) wc->tris++;
            if (mt_hit(ox, oy, oz, dx, dy, dz, a, b, c, tmin, tmax, t)) return true;
        }
        return false;
    }
    RayBox rb = make_raybox(ox, oy, oz, dx, dy, dz);
    int sp = 0;
    int node = s.root;
    while (true) {
        if (node >= 0) {
            if (CNT) wc->nodes++;
            const float4* nd = s.nodes + 4 * node;
            float4 n0 = nd[0], n1 = nd[1], n2 = nd[2], n3 = nd[3];
            float tl, tr;
            bool hl = slab(rb, n0, n1, tmin, tmax, tl);
            bool hr = slab(rb, n2, n3, tmin, tmax, tr);
            int cl = __float_as_int(n0.w), cr = __float_as_int(n1.w);
            if (hl && hr) {
                stack[sp * stride] = cr;
                ++sp;
                node = cl;
                continue;
            } else if (hl) {
                node = cl;
                continue;
            } else if (hr) {
                node = cr;
                continue;
            }
        } else {
            int i = ~node;
            float4 a = s.tri4[3 * i], b = s.tri4[3 * i + 1], c = s.tri4[3 * i + 2];
            int sf = __float_as_int(b.w);
            float t;
            if (CNT && sf != skip_a && sf != skip_b) wc->tris++;
            if (sf != skip_a && sf != skip_b &&
                mt_hit(ox, oy, oz, dx, dy, dz, a, b, c, tmin, tmax, t))
                return true;
        }
        if (sp == 0) break;
        --sp;
        node = stack[sp * stride];
    }
    return false;
}

// Leg A -> B blocked?  FP32 ray from fl(A) along fl((B - A) x (1 / L)), EPS < t < L - EPS,
// ignoring the surfaces sa, sb of its end points.
template <bool BRUTE, bool CNT = false>
__device__ bool leg_blocked(const SceneView& s, const double* A, const double* B, int sa, int sb,
                            int* stack, int stride, WorkCount* wc = nullptr)
{
#pragma clang fp contract(off)
    double w0 = B[0] - A[0], w1 = B[1] - A[1], w2 = B[2] - A[2];
    double L, il;
    sqrt_inv(w0 * w0 + w1 * w1 + w2 * w2, L, il);
    float tmin = (float)RT_EPS;
    float tmax = (float)(L - RT_EPS);
    if (!(tmax > tmin)) return false;
    return any_hit<BRUTE, CNT>(s, (float)A[0], (float)A[1], (float)A[2], (float)(w0 * il), (float)(w1 * il),
                               (float)(w2 * il), tmin, tmax, sa, sb, stack, stride, wc);
}

// --------------------------------------------------------------------------
// Wave-coherent any hit.  The lanes of one wave walk the BVH together: a
// child is entered when its box test succeeds for any lane still searching;
// node index and stack are wave-uniform (one LDS stack per wave).  Each lane
// tests its own ray against every leaf reached, so its answer is exactly the
// per-lane any-hit answer (which does not depend on the nodes visited).
// Call from wave-uniform control flow; `searching` masks lanes out.
// --------------------------------------------------------------------------
template <bool CNT>
__device__ bool any_hit_wave(const SceneView& s, bool searching, float ox, float oy, float oz, float dx, float dy,
                             float dz, float tmin, float tmax, int skip_a, int skip_b, int* wstack,
                             WorkCount* wc)
{
    bool hit = false;
    if (s.n_tri == 0 || __ballot(searching) == 0ull) return false;
    RayBox rb = make_raybox(ox, oy, oz, dx, dy, dz);
    int sp = 0;
    int node = s.root;
    while (true) {
        if (node >= 0) {
            const float4* nd = s.nodes + 4 * node;
            float4 n0 = nd[0], n1 = nd[1], n2 = nd[2], n3 = nd[3];
            float tl, tr;
            bool hl = searching && slab(rb, n0, n1, tmin, tmax, tl);
            bool hr = searching && slab(rb, n2, n3, tmin, tmax, tr);
            const unsigned long long bl = __ballot(hl), br = __ballot(hr);
            const int cl = __builtin_amdgcn_readfirstlane(__float_as_int(n0.w));
            const int cr = __builtin_amdgcn_readfirstlane(__float_as_int(n1.w));
            if (CNT) {
                if (hl && cl >= 0) wc->nodes++;
                if (hr && cr >= 0) wc->nodes++;
            }
            if (bl && br) {
                wstack[sp] = cr;
                ++sp;
                node = cl;
                continue;
            } else if (bl) {
                node = cl;
                continue;
            } else if (br) {
                node = cr;
                continue;
            }
        } else {
            const int i = ~node;
            float4 a = s.tri4[3 * i], b = s.tri4[3 * i + 1], c = s.tri4[3 * i + 2];
            const int sf = __float_as_int(b.w);
            if (sf != skip_a && sf != skip_b && searching) {
                float t;
                if (CNT) wc->tris++;
                if (mt_hit(ox, oy, oz, dx, dy, dz, a, b, c, tmin, tmax, t)) {
                    hit = true;
                    searching = false;
                }
            }
            if (__ballot(searching) == 0ull) break;
        }
        if (sp == 0) break;
        --sp;
        node = __builtin_amdgcn_readfirstlane(wstack[sp]);
    }
    return hit;
}

// 4-wide collapse of the binary tree, used by the wave-coherent walk: the
// node of every internal node n of even depth lists the grandchildren of n
// (or a child itself where that child is a leaf), with the boxes the binary
// nodes hold, so the boxes and the conservativeness of the test are the same.
// Layout per node (8 float4): lo.x, hi.x, lo.y, hi.y, lo.z, hi.z of the four
// entries, the four references (>= 0 node, < 0 ~leaf slot, RT_NODE4_EMPTY
// unused), and the surface of each leaf entry (-1 otherwise).  Node indices are those of the binary tree.  An
// unused entry has a zero box and is masked out by its reference.
#define RT_NODE4_EMPTY 0x7fffffff
#define RT_STACK4 (3 * (RT_STACK / 2) + 4)

__device__ __forceinline__ bool slab1(float lx, float hx, float ly, float hy, float lz, float hz, const RayBox& r,
                                      float tmin, float tmax)
{
    float t0x = __builtin_fmaf(lx, r.ix, -r.oix), t1x = __builtin_fmaf(hx, r.ix, -r.oix);
    float t0y = __builtin_fmaf(ly, r.iy, -r.oiy), t1y = __builtin_fmaf(hy, r.iy, -r.oiy);
    float t0z = __builtin_fmaf(lz, r.iz, -r.oiz), t1z = __builtin_fmaf(hz, r.iz, -r.oiz);
    float a = fmaxf(fmaxf(fminf(t0x, t1x), fminf(t0y, t1y)), fmaxf(fminf(t0z, t1z), tmin));
    float b = fminf(fminf(fmaxf(t0x, t1x), fmaxf(t0y, t1y)), fminf(fmaxf(t0z, t1z), tmax));
    return a <= b;
}

// any_hit_wave over the 4-wide nodes (same answer per lane).  `wstack` holds
// RT_STACK4 entries for the wave.
__device__ bool any_hit_wave4(const SceneView& s, bool searching, float ox, float oy, float oz, float dx, float dy,
                              float dz, float tmin, float tmax, int skip_a, int skip_b, int* wstack)
{
    bool hit = false;
    if (s.n_tri == 0 || __ballot(searching) == 0ull) return false;
    const RayBox rb = make_raybox(ox, oy, oz, dx, dy, dz);
    int sp = 0;
    int node = s.root;
    while (true) {
        if (node >= 0) {
            const float4* q = s.node4 + 8 * node;
            const float4 lx = q[0], hx = q[1], ly = q[2], hy = q[3], lz = q[4], hz = q[5], cf = q[6], sfs = q[7];
            const int c0 = __float_as_int(cf.x), c1 = __float_as_int(cf.y);
            const int c2 = __float_as_int(cf.z), c3 = __float_as_int(cf.w);
            // unused entries and leaves of an ignored surface are masked after the ballot, without a branch
            const int f0 = __float_as_int(sfs.x), f1 = __float_as_int(sfs.y);
            const int f2 = __float_as_int(sfs.z), f3 = __float_as_int(sfs.w);
            const unsigned long long m0 = __ballot(slab1(lx.x, hx.x, ly.x, hy.x, lz.x, hz.x, rb, tmin, tmax) & searching) &
                                          ((f0 >= 0 && (f0 == skip_a || f0 == skip_b)) ? 0ull : ~0ull);
            const unsigned long long m1 = __ballot(slab1(lx.y, hx.y, ly.y, hy.y, lz.y, hz.y, rb, tmin, tmax) & searching) &
                                          ((f1 >= 0 && (f1 == skip_a || f1 == skip_b)) ? 0ull : ~0ull);
            const unsigned long long m2 = __ballot(slab1(lx.z, hx.z, ly.z, hy.z, lz.z, hz.z, rb, tmin, tmax) & searching) &
                                          ((c2 == RT_NODE4_EMPTY || (f2 >= 0 && (f2 == skip_a || f2 == skip_b))) ? 0ull : ~0ull);
            const unsigned long long m3 = __ballot(slab1(lx.w, hx.w, ly.w, hy.w, lz.w, hz.w, rb, tmin, tmax) & searching) &
                                          ((c3 == RT_NODE4_EMPTY || (f3 >= 0 && (f3 == skip_a || f3 == skip_b))) ? 0ull : ~0ull);
            // visit the first entry hit, push the others (last pushed = next visited)
            int next = RT_NODE4_EMPTY;
            if (m3) next = c3;
            if (m2) {
                if (next != RT_NODE4_EMPTY) wstack[sp++] = next;
                next = c2;
            }
            if (m1) {
                if (next != RT_NODE4_EMPTY) wstack[sp++] = next;
                next = c1;
            }
            if (m0) {
                if (next != RT_NODE4_EMPTY) wstack[sp++] = next;
                next = c0;
            }
            if (next != RT_NODE4_EMPTY) {
                node = next;
                continue;
            }
        } else {
            const int i = ~node;
            float4 a = s.tri4[3 * i], b = s.tri4[3 * i + 1], c = s.tri4[3 * i + 2];
            const int sf = __float_as_int(b.w);
            if (sf != skip_a && sf != skip_b && searching) {
                float t;
                if (mt_hit(ox, oy, oz, dx, dy, dz, a, b, c, tmin, tmax, t)) {
                    hit = true;
                    searching = false;
                }
            }
            if (__ballot(searching) == 0ull) break;
        }
        if (sp == 0) break;
        --sp;
        node = __builtin_amdgcn_readfirstlane(wstack[sp]);
    }
    return hit;
}

__device__ __forceinline__ bool slab1t(float lx, float hx, float ly, float hy, float lz, float hz, const RayBox& r,
                                       float tmin, float tmax, float& tn)
{
    float t0x = __builtin_fmaf(lx, r.ix, -r.oix), t1x = __builtin_fmaf(hx, r.ix, -r.oix);
    float t0y = __builtin_fmaf(ly, r.iy, -r.oiy), t1y = __builtin_fmaf(hy, r.iy, -r.oiy);
    float t0z = __builtin_fmaf(lz, r.iz, -r.oiz), t1z = __builtin_fmaf(hz, r.iz, -r.oiz);
    float a = fmaxf(fmaxf(fminf(t0x, t1x), fminf(t0y, t1y)), fmaxf(fminf(t0z, t1z), tmin));
    float b = fminf(fminf(fmaxf(t0x, t1x), fmaxf(t0y, t1y)), fminf(fmaxf(t0z, t1z), tmax));
    tn = a;
    return a <= b;
}

// Closest hit for a wave: the lanes walk the 4-wide nodes together (node
// data in scalar registers), each lane pruning boxes with its own best
// distance; the entries of a node are visited nearest first as seen by the
// first searching lane.  A lane's answer is the lowest (t, triangle id) over
// every triangle but skip_tri with tmin < t, as in closest_hit: a triangle
// is tested by every lane whenever some lane's ray reaches its box, and a
// lane only prunes boxes it cannot improve on.  wstack: RT_STACK4 entries.
__device__ int closest_hit_wave4(const SceneView& s, bool active, float ox, float oy, float oz, float dx, float dy,
                                 float dz, float tmin, int skip_tri, int* wstack, float& t_best, int& id_best)
{
    const float inf = __builtin_inff();
    t_best = inf;
    id_best = 0x7fffffff;
    int slot_best = -1;
    const unsigned long long act = __ballot(active);
    if (s.n_tri == 0 || act == 0ull) return -1;
    const int lead = __ffsll((long long)act) - 1;
    const RayBox rb = make_raybox(ox, oy, oz, dx, dy, dz);
    int sp = 0;
    int node = s.root;
    while (true) {
        if (node >= 0) {
            const float4* q = s.node4 + 8 * node;
            const float4 lx = q[0], hx = q[1], ly = q[2], hy = q[3], lz = q[4], hz = q[5], cf = q[6];
            int c0 = __float_as_int(cf.x), c1 = __float_as_int(cf.y);
            int c2 = __float_as_int(cf.z), c3 = __float_as_int(cf.w);
            float t0, t1, t2, t3;
            const bool h0 = slab1t(lx.x, hx.x, ly.x, hy.x, lz.x, hz.x, rb, tmin, t_best, t0) & active;
            const bool h1 = slab1t(lx.y, hx.y, ly.y, hy.y, lz.y, hz.y, rb, tmin, t_best, t1) & active;
            const bool h2 = slab1t(lx.z, hx.z, ly.z, hy.z, lz.z, hz.z, rb, tmin, t_best, t2) & active;
            const bool h3 = slab1t(lx.w, hx.w, ly.w, hy.w, lz.w, hz.w, rb, tmin, t_best, t3) & active;
            const bool v0 = __ballot(h0) != 0ull, v1 = __ballot(h1) != 0ull;
            const bool v2 = c2 != RT_NODE4_EMPTY && __ballot(h2) != 0ull;
            const bool v3 = c3 != RT_NODE4_EMPTY && __ballot(h3) != 0ull;
            // sort keys: the lead lane's entry distance; entries it misses after those it hits,
            // entries no lane hits (dropped) last
            const float big = 3.0e38f;
            float k0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(h0 ? t0 : big), lead));
            float k1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(h1 ? t1 : big), lead));
            float k2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(h2 ? t2 : big), lead));
            float k3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(h3 ? t3 : big), lead));
            k0 = v0 ? k0 : inf;
            k1 = v1 ? k1 : inf;
            k2 = v2 ? k2 : inf;
            k3 = v3 ? k3 : inf;
            c0 = v0 ? c0 : RT_NODE4_EMPTY;
            c1 = v1 ? c1 : RT_NODE4_EMPTY;
            c2 = v2 ? c2 : RT_NODE4_EMPTY;
            c3 = v3 ? c3 : RT_NODE4_EMPTY;
#define RT_CSWAP(ka, ca, kb, cb)                  \
    {                                             \
        const bool sw = kb < ka;                  \
        const float tk = sw ? kb : ka;            \
        kb = sw ? ka : kb;                        \
        ka = tk;                                  \
        const int tc = sw ? cb : ca;              \
        cb = sw ? ca : cb;                        \
        ca = tc;                                  \
    }
            RT_CSWAP(k0, c0, k1, c1)
            RT_CSWAP(k2, c2, k3, c3)
            RT_CSWAP(k0, c0, k2, c2)
            RT_CSWAP(k1, c1, k3, c3)
            RT_CSWAP(k1, c1, k2, c2)
#undef RT_CSWAP
            // the order is wave-uniform: keep it in scalar registers
            c0 = __builtin_amdgcn_readfirstlane(c0);
            c1 = __builtin_amdgcn_readfirstlane(c1);
            c2 = __builtin_amdgcn_readfirstlane(c2);
            c3 = __builtin_amdgcn_readfirstlane(c3);
            if (c3 != RT_NODE4_EMPTY) wstack[sp++] = c3;
            if (c2 != RT_NODE4_EMPTY) wstack[sp++] = c2;
            if (c1 != RT_NODE4_EMPTY) wstack[sp++] = c1;
            if (c0 != RT_NODE4_EMPTY) {
                node = c0;
                continue;
            }
        } else {
            const int i = ~node;
            const float4 a = s.tri4[3 * i], b = s.tri4[3 * i + 1], c = s.tri4[3 * i + 2];
            const int id = __float_as_int(a.w);
            if (active && id != skip_tri) {
                float t;
                if (mt_hit(ox, oy, oz, dx, dy, dz, a, b, c, tmin, inf, t)) {
                    if (t < t_best || (t == t_best && id < id_best)) {
                        t_best = t;
                        id_best = id;
                        slot_best = i;
                    }
                }
            }
        }
        if (sp == 0) break;
        --sp;
        node = __builtin_amdgcn_readfirstlane(wstack[sp]);
    }
    return slot_best;
}

// v of a quad's four lanes, or-ed (quad_perm [1,0,3,2], then [2,3,0,1])
__device__ __forceinline__ int quad_or(int v)
{
    v |= __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);
    return v | __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);
}

// Closest hit with four lanes per ray, lane e of a quad testing entry e of the
// 4-wide node its ray is at (16 rays walk on their own in a wave).  A leaf
// entry that is hit is tested at once, the four of a node side by side; the
// inner entries that are hit are ordered by distance within the quad, the
// nearest is visited next and the others wait on the quad's stack in LDS with
// their distances (entries that the best hit has passed are dropped unvisited).
// For rays too sparse to share nodes, where closest_hit_wave4 visits the union
// of 64 rays' nodes.  The answer is the same: the lowest (t, triangle id) over
// every triangle but skip_tri with tmin < t; the same on the four lanes.
// st: this quad's stack, `stride` int2 between its entries.
__device__ __forceinline__ int closest_hit_quad(const SceneView& s, bool active, float ox, float oy, float oz,
                                                float dx, float dy, float dz, float tmin, int skip_tri, int2* st,
                                                int stride, float& t_best, int& id_best)
{
    const float inf = __builtin_inff();
    const int e = threadIdx.x & 3;
    t_best = inf;
    id_best = 0x7fffffff;
    int slot_best = -1;
    // a leaf entry's triangle, then the best of the quad
    auto leaf = [&](bool test, int slot) {
        float t = inf;
        int id = 0x7fffffff;
        if (test) {
            const float4* tp = s.tri4 + 3 * (int64_t)slot;
            const float4 a = tp[0], b = tp[1], c = tp[2];
            id = __float_as_int(a.w);
            float th;
            if (id != skip_tri && mt_hit(ox, oy, oz, dx, dy, dz, a, b, c, tmin, inf, th))
                t = th;
            else
                id = 0x7fffffff;
        }
        auto take = [&](float to, int ido, int so) {
            const bool better = to < t || (to == t && ido < id);
            t = better ? to : t;
            id = better ? ido : id;
            slot = better ? so : slot;
        };
        take(__int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(t), 0xB1, 0xF, 0xF, true)),
             __builtin_amdgcn_update_dpp(0, id, 0xB1, 0xF, 0xF, true),
             __builtin_amdgcn_update_dpp(0, slot, 0xB1, 0xF, 0xF, true));
        take(__int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(t), 0x4E, 0xF, 0xF, true)),
             __builtin_amdgcn_update_dpp(0, id, 0x4E, 0xF, 0xF, true),
             __builtin_amdgcn_update_dpp(0, slot, 0x4E, 0xF, 0xF, true));
        if (t < t_best || (t == t_best && id < id_best)) {
            t_best = t;
            id_best = id;
            slot_best = slot;
        }
    };
    if (s.n_tri == 0) return -1;
    if (s.root < 0) {
        leaf(active && e == 0, ~s.root);
        return slot_best;
    }
    const RayBox rb = make_raybox(ox, oy, oz, dx, dy, dz);
    int node = s.root, sp = 0;
    bool walking = active;
    while (__ballot(walking) != 0ull) {
        bool hit = false, inner = false;
        int ref = 0;
        float tn = inf;
        if (walking) {
            const float* q = (const float*)(s.node4 + 8 * (int64_t)node) + e;
            ref = __float_as_int(q[24]);
            hit = slab1t(q[0], q[4], q[8], q[12], q[16], q[20], rb, tmin, t_best, tn) && ref != RT_NODE4_EMPTY;
        }
        if (__ballot(hit && ref < 0) != 0ull) leaf(hit && ref < 0, ~ref);
        inner = hit && ref >= 0 && tn <= t_best;
        // rank among the quad's inner hits by (distance, entry)
        const int k = inner ? __float_as_int(tn) : 0x7f800000;   // distances are positive: bits order as they do
        const int k0 = __builtin_amdgcn_update_dpp(0, k, 0x00, 0xF, 0xF, true);
        const int k1 = __builtin_amdgcn_update_dpp(0, k, 0x55, 0xF, 0xF, true);
        const int k2 = __builtin_amdgcn_update_dpp(0, k, 0xAA, 0xF, 0xF, true);
        const int k3 = __builtin_amdgcn_update_dpp(0, k, 0xFF, 0xF, 0xF, true);
        const int rank = (k0 < k || (k0 == k && 0 < e)) + (k1 < k || (k1 == k && 1 < e)) +
                         (k2 < k || (k2 == k && 2 < e)) + (k3 < k);
        const int n = (k0 < 0x7f800000) + (k1 < 0x7f800000) + (k2 < 0x7f800000) + (k3 < 0x7f800000);
        if (inner && rank > 0) st[(sp + n - 1 - rank) * stride] = make_int2(ref, k);
        const int near = quad_or(inner && rank == 0 ? ref : 0);
        if (walking) {
            node = near;
            sp += n > 0 ? n - 1 : 0;
            if (n == 0) {   // nothing below: the nearest waiting entry that the best hit has not passed
                walking = false;
                while (sp > 0) {
                    const int2 top = st[--sp * stride];
                    if (__int_as_float(top.y) <= t_best) {
                        node = top.x;
                        walking = true;
                        break;
                    }
                }
            }
        }
    }
    return slot_best;
}

// --------------------------------------------------------------------------
// Tube walk for a wave of nearly parallel segments (the legs of one slot for
// 64 RIS elements).  Every lane's tested segment o + t d, t in [tmin, tmax],
// lies within r of the central segment cA -> cB (the distance between points
// of equal parameter is at most the larger end-point distance), so a
// triangle the lane's own test can accept has its (inflated) leaf box within
// r of the central segment.  The wave walks the 4-wide nodes breadth first
// with only the central segment against boxes grown by r (+ a margin for the
// FP32 representation of the lanes' rays, the triangle test and the slab
// test), one entry per lane, collecting candidate leaves; then every lane
// tests its own ray against the candidates with the exact triangle test.
// The result per lane is the any-hit answer of the lane's ray (a superset of
// the triangles it could hit is tested with the same test).  If the frontier
// or the candidate list outgrows its LDS space, the wave falls back to the
// 4-wide wave walk.
// --------------------------------------------------------------------------
#define RT_TUBE_FRONT 128
#define RT_TUBE_CAND 128

// Maximum over the 64 lanes of a wave (every lane active) of values >= 0 as
// their bits (a NaN comes out as the largest), with DPP lane moves: butterflies
// inside rows of 16, then the row broadcasts of the 64-wide wave; lane 63 ends
// with the maximum.
__device__ __forceinline__ float wave_max_pos(float v)
{
    unsigned x = __float_as_uint(v);
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true));
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true));
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xF, 0xF, true));
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xF, 0xF, true));
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false));
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false));
    return __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)x, 63));
}

// Maximum over the 64 lanes of a wave (every lane active), with DPP lane
// moves: butterflies inside rows of 16, then the row broadcasts of the
// 64-wide wave; lane 63 ends with the maximum.
__device__ __forceinline__ float wave_max(float v)
{
    int x = __float_as_int(v);
    x = __float_as_int(fmaxf(__int_as_float(x), __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false))));
    x = __float_as_int(fmaxf(__int_as_float(x), __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false))));
    x = __float_as_int(fmaxf(__int_as_float(x), __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0x124, 0xF, 0xF, false))));
    x = __float_as_int(fmaxf(__int_as_float(x), __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0x128, 0xF, 0xF, false))));
    x = __float_as_int(fmaxf(__int_as_float(x), __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0x142, 0xA, 0xF, false))));
    x = __float_as_int(fmaxf(__int_as_float(x), __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0x143, 0xC, 0xF, false))));
    return __int_as_float(__builtin_amdgcn_readlane(x, 63));
}

// All legs of one slot at once: one tube per leg, frontier and candidate
// entries tagged with their leg (3 bits above a 29-bit node or slot index),
// so the wave walks the levels of the tree once for up to KM + 1 legs.
// legs: the lanes' rays; end: the last leg's end point (the receiver, the same
// for every lane); tube: 3 float4 per leg in LDS; front: 2 x RT_TUBE_FRONT
// ints (the fallback's stack as well), cand: RT_TUBE_CAND ints, all per wave;
// seq: the slot's surfaces (wave-uniform), k its order; ok: the lane's path
// is still valid.  Returns the lane's bit set of blocked legs, plus
// RT_TUBE_FELL_BACK if the lists overflowed and the legs were walked one by
// one.
#define RT_TUBE_FELL_BACK 256u
#define RT_TUBE_TAG_SHIFT 29
#define RT_TUBE_IDX_MASK 0x1fffffffu
// a frontier or candidate entry: node or leaf slot index (< 2^29) and leg j (3 bits), as int
__device__ __forceinline__ int tube_entry(int idx, int j)
{
    return (int)((unsigned)idx | ((unsigned)j << RT_TUBE_TAG_SHIFT));
}
// surface at the start (a) or end (b) of leg j of a slot of order k (-1: a
// source or receiver), selected by value (j differs between lanes)
template <int KM>
__device__ __forceinline__ int leg_surface_a(const int* seq, int j)
{
    int v = -1;
#pragma unroll
    for (int q = 0; q < KM; ++q) v = (j == q + 1) ? seq[q] : v;
    return v;
}
template <int KM>
__device__ __forceinline__ int leg_surface_b(const int* seq, int j, int k)
{
    int v = -1;
#pragma unroll
    for (int q = 0; q < KM; ++q) v = (j == q && j != k) ? seq[q] : v;
    return v;
}

// A lane's leg rays, 7 floats each: ox, oy, oz, dx, dy, dz, tmax.  The first
// REG legs in registers, the others in the wave's part of LDS, [leg][7][64].
// LDS is given out in 1280 bytes of a CU's 160 KB: with two of six legs in registers
// four waves fit a SIMD (three without), with one of four five (four without).
template <int KM>
struct LegRays {
    static constexpr int REG = KM > RT_KM_SMALL ? 2 : 1;
    static constexpr int LDS_FLOATS = (KM + 1 - REG) * 7 * 64;   // per wave
    float reg[REG > 0 ? REG : 1][7];
    float* lds;   // this lane's first
    // j, c: constants
    __device__ __forceinline__ void set(int j, int c, float v)
    {
        if (j < REG)
            reg[j < REG ? j : 0][c] = v;
        else
            lds[((j - REG) * 7 + c) * 64] = v;
    }
    __device__ __forceinline__ float at(int j, int c) const
    {
        return j < REG ? reg[j < REG ? j : 0][c] : lds[((j - REG) * 7 + c) * 64];
    }
    // leg j, the same for every lane of the wave
    __device__ __forceinline__ void get(int j, float* r) const
    {
        if (j < REG) {
#pragma unroll
            for (int c = 0; c < 7; ++c) r[c] = j == 0 ? reg[0][c] : reg[REG > 1 ? 1 : 0][c];
        } else {
#pragma unroll
            for (int c = 0; c < 7; ++c) r[c] = lds[((j - REG) * 7 + c) * 64];
        }
    }
};

template <int KM>
__device__ __forceinline__ unsigned legs_blocked_tube(const SceneView& s, bool ok, int k, const int* seq,
                                                      const LegRays<KM>& legs, const float* end, float4* tube,
                                                      int* front, int* cand)
{
    static_assert(KM + 1 <= 8, "three bits of leg index");
    static_assert(2 * RT_TUBE_FRONT >= RT_STACK4, "the fallback's stack");
    const int lane = threadIdx.x & 63;
    const float tmin = (float)RT_EPS;
    unsigned blocked = 0;
    if (s.n_tri == 0 || __ballot(ok) == 0ull) return 0;
    // Path vertices of the first valid lane (the central path) and the largest
    // distance of any lane's from them, vertex j in lane j: per vertex one wave
    // maximum of squares; the tubes' constants follow in lanes 0..k at once.
    // (Per leg, with both end points, square roots and constants computed by
    // every lane, the set-up took 75 vector instructions a leg; 30 so, and 45 a
    // slot.)
    const int lead = __ffsll((long long)__ballot(ok)) - 1;
    unsigned live = 0;   // legs with a searching lane (uniform)
    float vx = 0.0f, vy = 0.0f, vz = 0.0f, vd = 0.0f;
#pragma unroll
    for (int j = 0; j <= KM + 1; ++j) {
        if (j > k + 1) break;
        float cx, cy, cz, d2 = 0.0f;
        if (j <= k) {
            const int jc = j <= KM ? j : KM;
            const float ox = legs.at(jc, 0), oy = legs.at(jc, 1), oz = legs.at(jc, 2);
            live |= __ballot(ok && legs.at(jc, 6) > tmin) ? 1u << j : 0u;
            cx = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ox), lead));
            cy = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(oy), lead));
            cz = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(oz), lead));
            const float ax = ox - cx, ay = oy - cy, az = oz - cz;
            d2 = wave_max_pos(ok ? __builtin_fmaf(ax, ax, __builtin_fmaf(ay, ay, az * az)) : 0.0f);
        } else {
            cx = end[0];
            cy = end[1];
            cz = end[2];
        }
        vx = lane == j ? cx : vx;
        vy = lane == j ? cy : vy;
        vz = lane == j ? cz : vz;
        vd = lane == j ? d2 : vd;
    }
    if (live == 0) return 0;
    bool overflow;
    {
        // the leg's end: the next lane's vertex (row_shl:1)
        const float wx = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(vx), 0x101, 0xF, 0xF, true));
        const float wy = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(vy), 0x101, 0xF, 0xF, true));
        const float wz = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(vz), 0x101, 0xF, 0xF, true));
        const float wd = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(vd), 0x101, 0xF, 0xF, true));
        float ex = wx - vx, ey = wy - vy, ez = wz - vz;
        // every lane's ray runs from its own vertex to its next one (direction and length in FP32): within the
        // larger of the two distances of the central leg, plus a margin for the FP32 representation of the rays,
        // the triangle test and the slab test: 1e-4 relative, 1e-4 m, 4e-6 of the coordinates' and leg's scale
        const float dev = __builtin_amdgcn_sqrtf(fmaxf(vd, wd));
        const float scale = fmaxf(fmaxf(fabsf(vx), fmaxf(fabsf(vy), fabsf(vz))),
                                  fmaxf(fabsf(wx), fmaxf(fabsf(wy), fabsf(wz)))) +
                            fabsf(ex) + fabsf(ey) + fabsf(ez) + 2.0f * dev;
        const float r = dev * 1.0002f + 1e-4f + 4e-6f * scale;
        // central ray with hardware reciprocals (1 ulp): their error is inside the margin too
        ex = fabsf(ex) < 1e-30f ? copysignf(1e-30f, ex) : ex;
        ey = fabsf(ey) < 1e-30f ? copysignf(1e-30f, ey) : ey;
        ez = fabsf(ez) < 1e-30f ? copysignf(1e-30f, ez) : ez;
        const float ix = __builtin_amdgcn_rcpf(ex), iy = __builtin_amdgcn_rcpf(ey), iz = __builtin_amdgcn_rcpf(ez);
        // a radius that is not representable: exact walk below
        overflow = __ballot(lane <= k && !(r < 1e30f)) != 0ull;
        if (lane <= k) {
            tube[3 * lane] = make_float4(ix, iy, iz, r);
            tube[3 * lane + 1] = make_float4(vx * ix, vy * iy, vz * iz,
                                             __int_as_float(leg_surface_a<KM>(seq, lane)));
            tube[3 * lane + 2].x = __int_as_float(leg_surface_b<KM>(seq, lane, k));
        }
    }
    int nc = 0;
    if (!overflow) {
        if (s.root < 0) {
            const int sf = __float_as_int(s.tri4[3 * (~s.root) + 1].w);
            for (int j = 0; j <= k; ++j)
                if ((live & (1u << j)) && sf != leg_surface_a<KM>(seq, j) && sf != leg_surface_b<KM>(seq, j, k)) {
                    if (lane == 0) cand[nc] = tube_entry(~s.root, j);
                    ++nc;
                }
        } else {
            int nf = 0, cur = 0;
            // The walk begins with the root's children, untested: the first round would test them with four
            // lanes a leg, the next one has room for 16 entries whether they passed or not (lab room 880 -> 815
            // us a launch, a room of 50000 triangles 930 -> 885).  A small scene's root, or one with a leaf
            // below it, goes first itself.
            static_assert(4 * (KM + 1) <= 64, "one lane per leg and child of the root");
            int rref = -1;
            if (s.n_tri >= 64) rref = __float_as_int(((const float*)(s.node4 + 8 * (int64_t)s.root))[24 + (lane & 3)]);
            if (__ballot(rref < 0) == 0ull) {
                const bool in = lane <= 4 * k + 3 && (live >> (lane >> 2) & 1u) && rref != RT_NODE4_EMPTY;
                const unsigned long long m = __ballot(in);
                if (in) front[__popcll(m & ((1ull << lane) - 1ull))] = tube_entry(rref, lane >> 2);
                nf = __popcll(m);
            } else {
                for (int j = 0; j <= k; ++j)
                    if (live & (1u << j)) {
                        if (lane == 0) front[nf] = tube_entry(s.root, j);
                        ++nf;
                    }
            }
            while (nf > 0) {
                int nn = 0;
                int* fin = front + cur * RT_TUBE_FRONT;
                int* fout = front + (cur ^ 1) * RT_TUBE_FRONT;
                for (int base = 0; base < nf; base += 16) {
                    const int slot = base + (lane >> 2), e = lane & 3;
                    const bool valid = slot < nf;
                    const unsigned v = valid ? (unsigned)fin[slot] : 0u;
                    const int n = (int)(v & RT_TUBE_IDX_MASK), j = (int)(v >> RT_TUBE_TAG_SHIFT);
                    const float4 t0 = tube[3 * j], t1 = tube[3 * j + 1];
                    RayBox crb;
                    crb.ix = t0.x;
                    crb.iy = t0.y;
                    crb.iz = t0.z;
                    crb.oix = t1.x;
                    crb.oiy = t1.y;
                    crb.oiz = t1.z;
                    const float r = t0.w;
                    const float* q = (const float*)(s.node4 + 8 * (int64_t)n);
                    const int ref = __float_as_int(q[24 + e]);
                    // a leaf of one of the leg's end-point surfaces is never a candidate of that leg
                    const int lsf = __float_as_int(q[28 + e]);
                    const bool skip = lsf >= 0 && (lsf == __float_as_int(t1.w) ||
                                                   lsf == __float_as_int(tube[3 * j + 2].x));
                    const bool hit = valid && ref != RT_NODE4_EMPTY && !skip &&
                                     slab1(q[e] - r, q[4 + e] + r, q[8 + e] - r, q[12 + e] + r, q[16 + e] - r,
                                           q[20 + e] + r, crb, -1e-3f, 1.001f);
                    const unsigned long long lt = (1ull << lane) - 1ull;
                    const unsigned long long mi = __ballot(hit && ref >= 0);
                    const unsigned long long ml = __ballot(hit && ref < 0);
                    if (hit && ref >= 0) {
                        const int idx = nn + __popcll(mi & lt);
                        if (idx < RT_TUBE_FRONT) fout[idx] = tube_entry(ref, j);
                    }
                    if (hit && ref < 0) {
                        const int idx = nc + __popcll(ml & lt);
                        if (idx < RT_TUBE_CAND) cand[idx] = tube_entry(~ref, j);
                    }
                    nn += __popcll(mi);
                    nc += __popcll(ml);
                }
                if (nn > RT_TUBE_FRONT || nc > RT_TUBE_CAND) {
                    overflow = true;
                    break;
                }
                nf = nn;
                cur ^= 1;
            }
        }
    }
    if (overflow) {   // exact walk of every leg
        blocked = RT_TUBE_FELL_BACK;
        for (int j = 0; j <= k; ++j) {
            float r[7];
            legs.get(j, r);
            const bool searching = ok && r[6] > tmin;
            const int sa = j == 0 ? -1 : seq[j - 1];
            const int sb = j == k ? -1 : seq[j];
            if (any_hit_wave4(s, searching, r[0], r[1], r[2], r[3], r[4], r[5], tmin, r[6], sa, sb, front))
                blocked |= 1u << j;
        }
        return blocked;
    }
    for (int i = 0; i < nc; ++i) {
        const unsigned v = (unsigned)__builtin_amdgcn_readfirstlane(cand[i]);
        const int slot = (int)(v & RT_TUBE_IDX_MASK), j = (int)(v >> RT_TUBE_TAG_SHIFT);
        const float4* tp = s.tri4 + 3 * (int64_t)slot;
        const float4 a = tp[0], b = tp[1], c = tp[2];
        float ray[7];
        legs.get(j, ray);
        const float ox = ray[0], oy = ray[1], oz = ray[2], dx = ray[3], dy = ray[4], dz = ray[5], tmax = ray[6];
        const bool open = ok && tmax > tmin && !(blocked & (1u << j));
        // most candidates are missed by every lane: decided without the division
        if (__ballot(open && mt_maybe(ox, oy, oz, dx, dy, dz, a, b, c)) == 0ull) continue;
        float t;
        if (open && mt_hit(ox, oy, oz, dx, dy, dz, a, b, c, tmin, tmax, t)) blocked |= 1u << j;
    }
    return blocked;
}

// --------------------------------------------------------------------------
// FP64 image method
// --------------------------------------------------------------------------
__device__ __forceinline__ double edge_raw(double sx, double sy, double ex, double ey, double px,
                                           double py)
{
#pragma clang fp contract(off)
    return (ex - sx) * (py - sy) - (ey - sy) * (px - sx);
}

// Edge function from the lexicographically smaller end point (exactly
// antisymmetric in the edge direction).
__device__ __forceinline__ double edge2(double sx, double sy, double ex, double ey, double px,
                                        double py)
{
    bool s_first = (sx < ex) || (sx == ex && sy < ey);
    return s_first ? edge_raw(sx, sy, ex, ey, px, py) : -edge_raw(ex, ey, sx, sy, px, py);
}

__device__ __forceinline__ bool top_left(double sx, double sy, double ex, double ey)
{
    double dy = ey - sy, dx = ex - sx;
    return (dy < 0.0) || (dy == 0.0 && dx < 0.0);
}

// Projection used by the containment test, computed once per triangle (same
// FP64 operations as a test that derives it on the fly): drop the axis of
// largest |normal| (lowest axis on ties), keep the other two in cyclic order,
// make the projected triangle counter-clockwise.  Writes 6 coordinates and
// the axes (16 if the projected area is 0: such a triangle contains nothing).
__device__ inline void triangle_projection(const double* v, double* out, int32_t* axes)
{
#pragma clang fp contract(off)
    double e1[3], e2[3];
    for (int k = 0; k < 3; ++k) {
        e1[k] = v[3 + k] - v[k];
        e2[k] = v[6 + k] - v[k];
    }
    double n0 = e1[1] * e2[2] - e1[2] * e2[1];
    double n1 = e1[2] * e2[0] - e1[0] * e2[2];
    double n2 = e1[0] * e2[1] - e1[1] * e2[0];
    double ax = fabs(n0), ay = fabs(n1), az = fabs(n2);
    int drop = 0;
    if (ay > ax && ay >= az) drop = 1;
    else if (az > ax && az > ay) drop = 2;
    int i0 = (drop + 1) % 3, i1 = (drop + 2) % 3;
    double a0 = v[i0], a1 = v[i1];
    double b0 = v[3 + i0], b1 = v[3 + i1];
    double c0 = v[6 + i0], c1 = v[6 + i1];
    double area = edge2(a0, a1, b0, b1, c0, c1);
    if (area < 0.0) {
        double t0 = b0, t1 = b1;
        b0 = c0; b1 = c1;
        c0 = t0; c1 = t1;
    }
    out[0] = a0; out[1] = a1; out[2] = b0; out[3] = b1; out[4] = c0; out[5] = c1;
    *axes = (area == 0.0) ? 16 : (i0 | (i1 << 2));
}

// Edge functions of the containment test, from the projection: per edge the
// lexicographically smaller end point and the edge vector from it, negated
// where the test negates (exact either way), so that one formula
//   w = dx (py - by) - dy (px - bx)
// gives the test's value.  The test is then three edge functions of five
// operations and a compare; derived from the vertices at every test it was some
// 75 vector instructions.
// [0] two integers, the axis the projection drops with the top-left edges in
// bits 2..4, and its axes as triangle_projection gives them; then per edge bx,
// by, dx, dy (dx = dy = 0 for a degenerate triangle: no value above 0).
__device__ inline void triangle_edges(const double* q6, int32_t axes, double* out)
{
#pragma clang fp contract(off)
    const int i0 = axes & 3;   // kept axes are drop + 1, drop + 2
    int32_t head[2] = {(i0 + 2) % 3, axes};
    const bool none = (axes & 16) != 0;
    for (int i = 0; i < 3; ++i) {
        // edges b c, c a, a b
        const int u = (i + 1) % 3, v = (i + 2) % 3;
        const double sx = q6[2 * u], sy = q6[2 * u + 1], ex = q6[2 * v], ey = q6[2 * v + 1];
        const bool s_first = (sx < ex) || (sx == ex && sy < ey);
        out[4 * i + 1] = s_first ? sx : ex;
        out[4 * i + 2] = s_first ? sy : ey;
        out[4 * i + 3] = none ? 0.0 : s_first ? ex - sx : -(sx - ex);
        out[4 * i + 4] = none ? 0.0 : s_first ? ey - sy : -(sy - ey);
        if (!none && top_left(sx, sy, ex, ey)) head[0] |= 4 << i;
    }
    __builtin_memcpy(&out[0], head, 8);
}

__device__ __forceinline__ int edge_axes(const double* t_edge, int t)
{
    return ((const int*)(t_edge + RT_EDGE * (int64_t)t))[1];
}

// p on the triangle's plane inside triangle t?  Half-open top-left rule in
// the triangle's projection: a point on an edge belongs to the triangle only
// if that edge is top-left, so a point on an edge shared by two coplanar
// triangles belongs to exactly one of them.
// UNIFORM: the same triangle for every lane of the wave, all its edges at once
// (scalar loads); else edge by edge, so that a lane whose point is outside the
// first reads half the record.
template <bool UNIFORM>
__device__ __forceinline__ bool contains_proj(const SceneView& s, int t, const double* p)
{
#pragma clang fp contract(off)
    const double* e = s.t_edge + RT_EDGE * (int64_t)t;
    const int head = ((const int*)e)[0], drop = head & 3;
    // what an edge's value has to exceed: 0, or the largest negative number (0 counts as inside)
    auto above = [head](int i) {
        const int tl = head >> (2 + i) & 1;
        return __hiloint2double(tl << 31, tl);
    };
    const double px = p[0], py = p[1], pz = p[2];
    const double q0 = drop == 0 ? py : drop == 1 ? pz : px;
    const double q1 = drop == 0 ? pz : drop == 1 ? px : py;
    const double w0 = e[3] * (q1 - e[2]) - e[4] * (q0 - e[1]);
    if (!UNIFORM && !(w0 > above(0))) return false;
    const double w1 = e[7] * (q1 - e[6]) - e[8] * (q0 - e[5]);
    const double w2 = e[11] * (q1 - e[10]) - e[12] * (q0 - e[9]);
    return w0 > above(0) && w1 > above(1) && w2 > above(2);
}

__device__ __forceinline__ double plane_side(const double* pl, const double* p)
{
#pragma clang fp contract(off)
    return (pl[0] * p[0] + pl[1] * p[1] + pl[2] * p[2]) - pl[3];
}

// Triangle of surface sf that contains p, or -1: the first in the
// surface's list.  With a grid, only the triangles listed for p's cell are
// tested, in list order: every triangle whose test could accept p overlaps
// that cell, so the answer is the same.  The counting build scans the whole
// list (the method's work).
template <bool CNT = false>
__device__ inline int surface_contains(const SceneView& s, int sf, const double* p, WorkCount* wc = nullptr)
{
    const double* bx = s.s_box + 6 * sf;
    const double px = p[0], py = p[1], pz = p[2];
    if (px < bx[0] || py < bx[1] || pz < bx[2] || px > bx[3] || py > bx[4] || pz > bx[5]) return -1;
    const int gax = CNT ? -1 : s.g_axes[sf];
    if (gax >= 0) {
        const double* fr = s.g_frame + 4 * sf;
        const int au = gax & 3, av = (gax >> 2) & 3, lg = gax >> 4;
        const double u = au == 0 ? px : au == 1 ? py : pz;
        const double v = av == 0 ? px : av == 1 ? py : pz;
        const int cell = (sgrid_index(u, fr[0], fr[2], lg) << lg) + sgrid_index(v, fr[1], fr[3], lg);
        const int64_t first = s.s_ptr[sf], b = RT_SGRID_CAP * first;
        const int32_t* off = s.g_off + RT_SGRID_OFF * first + sf + cell;
        const int end = off[1];
        for (int j = off[0]; j < end; ++j) {
            const int t = s.g_tris[b + j];
            if (contains_proj<false>(s, t, p)) return t;
        }
        return -1;
    }
    for (int j = s.s_ptr[sf]; j < s.s_ptr[sf + 1]; ++j) {
        int t = s.s_tris[j];
        if (CNT) wc->contain++;
        if (contains_proj<false>(s, t, p)) return t;
    }
    return -1;
}

// Mirror p in plane pl (n, c, n . n and its reciprocal): p - (2 side / n . n) n.
__device__ __forceinline__ void mirror(const double* pl, const double* p, double* out)
{
#pragma clang fp contract(off)
    const double f = div_by(2.0 * plane_side(pl, p), pl[4], pl[5]);
    out[0] = p[0] - f * pl[0];
    out[1] = p[1] - f * pl[1];
    out[2] = p[2] - f * pl[2];
}

// Back-trace from X through images I[1..k] (I[0] = source S) over surfaces
// seq; on success fills P[0..k) and tri[0..k).  The loops run over the
// compile-time bound KM >= k with constant indices so the arrays stay in
// registers.
template <int KM>
__device__ inline bool image_backtrace(const SceneView& s, const int* seq, int k, const double (*I)[3],
                                       const double* X, double (*P)[3], int* tri)
{
#pragma clang fp contract(off)
    double Q[3] = {X[0], X[1], X[2]};
#pragma unroll
    for (int i = KM; i >= 1; --i) {
        if (i > k) continue;
        const double* pl = s.s_plane + RT_PLANE * seq[i - 1];
        double w0 = Q[0] - I[i][0], w1 = Q[1] - I[i][1], w2 = Q[2] - I[i][2];
        double den = pl[0] * w0 + pl[1] * w1 + pl[2] * w2;
        if (den == 0.0) return false;
        double sp = div_fast(pl[3] - (pl[0] * I[i][0] + pl[1] * I[i][1] + pl[2] * I[i][2]), den);
        if (!(sp > 0.0 && sp < 1.0)) return false;
        double p[3] = {I[i][0] + sp * w0, I[i][1] + sp * w1, I[i][2] + sp * w2};
        int t = surface_contains(s, seq[i - 1], p);
        if (t < 0) return false;
        tri[i - 1] = t;
        P[i - 1][0] = p[0]; P[i - 1][1] = p[1]; P[i - 1][2] = p[2];
        Q[0] = p[0]; Q[1] = p[1]; Q[2] = p[2];
    }
#pragma unroll
    for (int i = 0; i < KM; ++i) {
        if (i >= k) break;
        const double* pl = s.s_plane + RT_PLANE * seq[i];
        double prev[3], next[3];
        for (int q = 0; q < 3; ++q) {
            prev[q] = i == 0 ? I[0][q] : P[i > 0 ? i - 1 : 0][q];
            next[q] = (i == k - 1 || i + 1 >= KM) ? X[q] : P[i + 1 < KM ? i + 1 : 0][q];
        }
        double a = plane_side(pl, prev);
        double b = plane_side(pl, next);
        if (!((a > 0.0 && b > 0.0) || (a < 0.0 && b < 0.0))) return false;
    }
    return true;
}

// --------------------------------------------------------------------------
// Patterns.  Whether a pattern factor is zero is decided on the FP64 cosine
// (cos^p: cos <= 0; monopole: sin(theta) = 0; isotropic: never), so that the
// decision does not depend on an underflow of the factor.  The amplitude
// factor sqrt(F) is evaluated directly in FP32: cos^(p/2), and the
// monopole's |cos(kh cos) - cos(kh)| / sin(theta) with sin^2 from FP64.
// --------------------------------------------------------------------------
__device__ __forceinline__ double cos_between(const double* v, const double* axis, double axis_norm)
{
    double n = sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    return (v[0] * axis[0] + v[1] * axis[1] + v[2] * axis[2]) / (n * axis_norm);
}

__device__ __forceinline__ bool pattern_on(int kind, double c)
{
    c = fmin(1.0, fmax(-1.0, c));
    if (kind == 0) return true;
    if (kind == 1) return c > 0.0;
    return 1.0 - c * c > 0.0;
}

__device__ __forceinline__ float pattern_amp(int kind, double param, double c64)
{
    c64 = fmin(1.0, fmax(-1.0, c64));
    if (kind == 0) return 1.0f;
    if (kind == 1) {   // 2^((p/2) log2 c) with the hardware's base-2 logarithm and exponential (1 ulp each)
        const float c = (float)c64;
        return c > 0.0f ? __builtin_amdgcn_exp2f((float)(0.5 * param) * __builtin_amdgcn_logf(c)) : 0.0f;
    }
    const double s2 = 1.0 - c64 * c64;   // sin^2(theta) in FP64: no cancellation to 0 near the axis
    if (!(s2 > 0.0)) return 0.0f;
    const float c = (float)c64, kh = (float)(6.283185307179586 * param);
    return fabsf(cosf(kh * c) - cosf(kh)) / sqrtf((float)s2);
}

// Gate and amplitude factor sqrt(F) of a pattern for the direction v against
// its axis.  For cos^p the gate (cos > 0) is the sign of v . axis, the
// cosine's numerator (the same decision as the FP64 cosine's sign: its
// denominator is positive), and the amplitude needs the cosine only in FP32;
// the monopole's gate needs the FP64 cosine itself; the isotropic pattern
// needs neither.
__device__ __forceinline__ bool pattern_gate_amp(int kind, double param, const double* v, const double* axis,
                                                 double axis_norm, float& amp)
{
    if (kind == 0) {
        amp = 1.0f;
        return true;
    }
    if (kind == 1) {
        const double dn = v[0] * axis[0] + v[1] * axis[1] + v[2] * axis[2];
        const float vv = (float)(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
        const float c = fminf(1.0f, (float)dn * __builtin_amdgcn_rsqf(vv) * __builtin_amdgcn_rcpf((float)axis_norm));
        amp = c > 0.0f ? __builtin_amdgcn_exp2f((float)(0.5 * param) * __builtin_amdgcn_logf(c)) : 0.0f;
        return dn > 0.0;
    }
    const double c = cos_between(v, axis, axis_norm);
    amp = pattern_amp(kind, param, c);
    return pattern_on(kind, c);
}

// e^{-j 2 pi d / lambda} = e^{-j 2 pi f}, f = frac(d / lambda) taken in FP64
// (d times 1 / lambda: a relative error of a few 1e-16 in turns); cosine and
// sine of the fraction of a turn by the hardware's v_cos/v_sin (their argument
// is in turns).
__device__ __forceinline__ void phase_cs(double d, double inv_lambda, float& cs, float& sn)
{
#pragma clang fp contract(off)
    const double x = d * inv_lambda;
    const float f = (float)(x - floor(x));
    cs = __builtin_amdgcn_cosf(f);
    sn = -__builtin_amdgcn_sinf(f);
}

// Fresnel reflection coefficient (Section II-B, specular reflection) of
// triangle t's material for a wave arriving along d (FP64): TE (pol 1)
//   (c - r) / (c + r), TM (pol 2) (eps c - r) / (eps c + r), r = sqrt(eps - 1 + c^2),
// c = |d . n| / |d| with n the unit normal of e1 x e2 from the FP64 vertices
// (precomputed per triangle) and len = |d| from the caller, eps = eps_r - j
// sigma sig_scale, principal square root (stable form for either sign of
// the real part).
__device__ inline float2 fresnel_coef(const SceneView& s, int t, const double* d, double len, int pol,
                                     double sig_scale)
{
#pragma clang fp contract(off)
    const double* nv = s.nrm + 3 * (int64_t)t;
    const double c = fmin(fabs(d[0] * nv[0] + d[1] * nv[1] + d[2] * nv[2]) / len, 1.0);   // len = |d|
    const float2 m = s.mat[t];
    const double er = (double)m.x, ei = -(double)m.y * sig_scale;
    const double a = er - (1.0 - c * c), b = ei;
    const double h = sqrt(a * a + b * b);
    double rr, ri;
    if (a >= 0.0) {
        rr = sqrt(0.5 * (h + a));
        ri = rr > 0.0 ? b / (2.0 * rr) : 0.0;
    } else {
        const double q = sqrt(0.5 * (h - a));
        rr = fabs(b) / (2.0 * q);
        ri = b < 0.0 ? -q : q;
    }
    double pr, pi, qr, qi;   // numerator p, denominator q
    if (pol == 1) {
        pr = c - rr; pi = -ri;
        qr = c + rr; qi = ri;
    } else {
        pr = er * c - rr; pi = ei * c - ri;
        qr = er * c + rr; qi = ei * c + ri;
    }
    const double iq = 1.0 / (qr * qr + qi * qi);
    return make_float2((float)((pr * qr + pi * qi) * iq), (float)((pi * qr - pr * qi) * iq));
}

// --------------------------------------------------------------------------
// launchers implemented in the .hip files
// --------------------------------------------------------------------------

}  // namespace rt
