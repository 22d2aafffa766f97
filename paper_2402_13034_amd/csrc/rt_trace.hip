// Tracing: discovery rays, candidate surface sequences, image-method paths,
// visibility legs, the per-element RIS expansion and the field.
//
// Stages (all on one stream; sizes are read back where buffers depend on them):
//  1. discovery  spherical-Fibonacci rays from the Tx (full sphere) and from
//                the RIS centre u (half-space in front of the RIS); closest
//                hit + specular bounce up to K times (stand-in for the
//                analytic first stage of the hybrid tracer, Section II).
//  2. dedupe     every prefix of every hit list, mapped to surfaces, packed
//                21 bits per surface into a key of one 64-bit word (orders
//                up to 3) or two (orders 4 and 5: surfaces 0-2 in word 0,
//                3-4 in word 1); hash set, then sort (+ unique for two words).
//  3. images     per candidate: images of the source in the surfaces' planes.
//  4. paths      per (receiver, candidate): image-method back-trace, surface
//                containment and side tests (FP64); the valid cells are
//                appended per wave and sorted into (receiver, candidate) order.
//  5. legs       each record's legs tested for occlusion (second stage of the
//                hybrid tracer; relaunch of Section IV-A).
//  6. field      Tx -> Rx: eq. (3) in the form of eq. (8) per path, summed per
//                receiver in record order (deterministic).
//  7. RIS        per (receiver, element): the direct element path and every
//                sequence valid from u re-run through the image method from
//                the element (Section II-B), legs re-checked, field of
//                eqs. (4)-(8) without Gamma summed into H[r, m].
#pragma clang fp contract(off)

#include <algorithm>
#include <cmath>
#include <cstring>
#include <exception>
#include <type_traits>
#include <memory>
#include <utility>
#include <vector>

#include "rt_host.hpp"

namespace rt {

static inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

__device__ __forceinline__ void wave_count_add(unsigned long long* ctr, unsigned v)
{
    // one atomic per wave
    unsigned long long s = v;
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0 && s) atomicAdd(ctr, s);
}

// Block-staged append: a block gathers its values in LDS (LDS atomics) and
// reserves room for all of them with one global atomic; values past `cap`
// are dropped while the counter keeps counting (the host checks it).  The
// order of the appended values is not fixed: callers sort them.
template <int NMAX>
struct BlockAppend {
    uint64_t* vals;   // LDS, NMAX entries
    int* n;           // LDS counter
    unsigned long long* base;   // LDS
    __device__ void init()
    {
        if (threadIdx.x == 0) *n = 0;
        __syncthreads();
    }
    __device__ void push(uint64_t v)
    {
        int slot = atomicAdd(n, 1);
        if (slot < NMAX) vals[slot] = v;
    }
    // every thread of the block must call flush
    __device__ void flush(uint64_t* out, int64_t cap, unsigned long long* counter)
    {
        __syncthreads();
        const int cnt = *n < NMAX ? *n : NMAX;
        if (threadIdx.x == 0) *base = cnt > 0 ? atomicAdd(counter, (unsigned long long)cnt) : 0ull;
        __syncthreads();
        for (int t = threadIdx.x; t < cnt; t += blockDim.x) {
            const unsigned long long idx = *base + (unsigned long long)t;
            if (idx < (unsigned long long)cap) out[idx] = vals[t];
        }
    }
};

// --------------------------------------------------------------------------
// 1. discovery
// --------------------------------------------------------------------------
__device__ __forceinline__ void fib_dir(int64_t i, int64_t n, double* out)
{
    const double g = (sqrt(5.0) - 1.0) / 2.0;
    double z = 1.0 - (double)(2 * i + 1) / (double)n;
    double x = (double)i * g;
    double ph = 6.283185307179586 * (x - floor(x));
    double r = sqrt(1.0 - z * z);
    out[0] = r * cos(ph);
    out[1] = r * sin(ph);
    out[2] = z;
}

constexpr int DISC_B = 128;


// Launch order of the discovery rows.  Consecutive Fibonacci rows form a
// thin band of directions (z falls linearly with the row); within a chunk of
// RT_FIB_CHUNK rows a wave should trace neighbouring azimuths.  The azimuth
// of row i0 + j is 2 pi frac(frac(i0 g) + frac(j g)), so the azimuth order of
// a chunk is one fixed order of j (by frac(j g)), rotated by an offset that
// depends on the chunk: position j of chunk c launches row
// c RT_FIB_CHUNK + perm[(off[c] + j) mod RT_FIB_CHUNK].  The tables are built
// once per context on the host; they only order the work (any order gives
// the same results).
#define RT_FIB_CHUNK 8192
#define RT_FIB_MAX_CHUNKS (((int64_t)1 << 31) / RT_FIB_CHUNK)

static void fib_tables(Ctx& c, const int32_t** perm, const int32_t** off)
{
    std::lock_guard<std::mutex> lk(c.fib_mu);
    if (!c.fib_perm) {
        const double g = (std::sqrt(5.0) - 1.0) / 2.0;
        std::vector<std::pair<double, int32_t>> fr(RT_FIB_CHUNK);
        for (int j = 0; j < RT_FIB_CHUNK; ++j) {
            const double x = (double)j * g;
            fr[j] = {x - std::floor(x), j};
        }
        std::sort(fr.begin(), fr.end());
        std::vector<int32_t> pm(RT_FIB_CHUNK), of((size_t)RT_FIB_MAX_CHUNKS);
        std::vector<double> fv(RT_FIB_CHUNK);
        for (int k = 0; k < RT_FIB_CHUNK; ++k) {
            pm[k] = fr[k].second;
            fv[k] = fr[k].first;
        }
        for (int64_t ch = 0; ch < RT_FIB_MAX_CHUNKS; ++ch) {
            const double x = (double)(ch * RT_FIB_CHUNK) * g;
            const double f0 = x - std::floor(x);
            of[(size_t)ch] = (int32_t)(std::lower_bound(fv.begin(), fv.end(), 1.0 - f0) - fv.begin()) % RT_FIB_CHUNK;
        }
        int32_t *dp = nullptr, *dofs = nullptr;
        HIP_CHECK(hipMalloc(&dp, sizeof(int32_t) * RT_FIB_CHUNK));
        HIP_CHECK(hipMalloc(&dofs, sizeof(int32_t) * (size_t)RT_FIB_MAX_CHUNKS));
        HIP_CHECK(hipMemcpy(dp, pm.data(), sizeof(int32_t) * RT_FIB_CHUNK, hipMemcpyHostToDevice));
        HIP_CHECK(hipMemcpy(dofs, of.data(), sizeof(int32_t) * (size_t)RT_FIB_MAX_CHUNKS, hipMemcpyHostToDevice));
        c.fib_perm = dp;
        c.fib_off = dofs;
    }
    *perm = c.fib_perm;
    *off = c.fib_off;
}

// Rows not launched keep -1 hit lists.
__global__ void k_fill_neg(int32_t* p, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = -1;
}

// De-duplication of prefix keys in an open-addressing hash set (keys != 0,
// capacity a power of two, linear probing; a probe run longer than max_probe
// raises the overflow flag, and the caller repeats with a larger set).  A slot is read before the
// compare-and-swap, so the many repeats of a key cost no atomics.
// mix64 is the 64-bit finalizer (fmix64) of Austin Appleby's public-domain
// MurmurHash3, constants as published.
__device__ __forceinline__ uint64_t mix64(uint64_t x)
{
    x ^= x >> 33;
    x *= 0xff51afd7ed558ccdull;
    x ^= x >> 33;
    x *= 0xc4ceb9fe1a85ec53ull;
    x ^= x >> 33;
    return x;
}

__device__ __forceinline__ void hash_insert(unsigned long long* table, uint64_t mask, uint64_t max_probe,
                                            uint64_t key, int* overflow)
{
    uint64_t h = mix64(key) & mask;
    for (uint64_t probe = 0; probe <= max_probe; ++probe) {
        // a plain read may be stale only as 0 (a slot changes once, 0 -> key); the CAS decides then
        unsigned long long cur = table[h];
        if (cur == key) return;
        if (cur == 0ull) {
            unsigned long long prev = atomicCAS(&table[h], 0ull, (unsigned long long)key);
            if (prev == 0ull || prev == key) return;
        }
        h = (h + 1) & mask;
    }
    atomicOr(overflow, 1);
}

// Two-word keys (orders 4 and 5): a slot is two words, word 0 (never 0 for a
// key: it holds the first surface) claimed by compare-and-swap, then word 1
// published with bit 63 set (0 = not yet written).  A lane that finds word 0
// equal to its key's but word 1 not (yet) equal probes on and may insert the
// key a second time; the sort that follows removes such duplicates, so a key
// is never lost and never kept twice.
#define RT_W1_SET (1ull << 63)
__device__ __forceinline__ void hash_insert2(unsigned long long* table, uint64_t mask, uint64_t max_probe,
                                             uint64_t k0, uint64_t k1, int* overflow)
{
    const unsigned long long w1 = (unsigned long long)(k1 | RT_W1_SET);
    uint64_t h = mix64(k0 ^ mix64(k1)) & mask;
    for (uint64_t probe = 0; probe <= max_probe; ++probe) {
        unsigned long long cur = table[2 * h];
        if (cur == 0ull) {
            const unsigned long long prev = atomicCAS(&table[2 * h], 0ull, (unsigned long long)k0);
            if (prev == 0ull) {
                atomicExch(&table[2 * h + 1], w1);
                return;
            }
            cur = prev;
        }
        if (cur == k0 && table[2 * h + 1] == w1) return;
        h = (h + 1) & mask;
    }
    atomicOr(overflow, 1);
}

// Discovery over the direction-sorted ray list; every prefix of every hit
// list (as surface ids) goes into the hash set.  Neighbouring lanes trace
// neighbouring directions, so a lane skips a key equal to its left
// neighbour's (one of them inserts it).  KM: the largest order of the
// instance (K <= KM); keys of orders above 3 have two words.
// CNT: the counting build: each lane walks the binary tree on its own (the
// method's per-ray LBVH walk, same hits) and the node visits, triangle tests
// and segments are added to work[0..2].
template <bool BRUTE, int STK, int KM, bool CNT>
__global__ __launch_bounds__(DISC_B) void k_discover(SceneView s, double sx, double sy, double sz,
                                                     const int32_t* perm, const int32_t* off, int64_t rows,
                                                     int hemi, double hx, double hy, double hz, int K,
                                                     int32_t* hits, unsigned long long* segs,
                                                     unsigned long long* table, uint64_t mask, uint64_t max_probe,
                                                     int* overflow, unsigned long long* work)
{
    constexpr int W = KM > RT_KM_SMALL ? 2 : 1;
    // per-lane stacks for the brute-force build and the counting build, one stack per wave for the wave walk
    __shared__ int stack[BRUTE ? 1 : (CNT ? STK * DISC_B : RT_STACK4 * (DISC_B / 64))];
    WorkCount wc;
    int64_t t = (int64_t)blockIdx.x * DISC_B + threadIdx.x;
    unsigned nseg = 0;
    uint64_t keys[KM], keys1[KM];   // key of each prefix: word 0, word 1
#pragma unroll
    for (int q = 0; q < KM; ++q) keys[q] = keys1[q] = 0ull;
    const int64_t ch = t / RT_FIB_CHUNK;
    const int64_t i = ch * RT_FIB_CHUNK + perm[(off[ch] + (int)(t % RT_FIB_CHUNK)) % RT_FIB_CHUNK];
    // the bounce loop runs for the whole wave; a lane drops out when its ray escapes
    double d64[3] = {0.0, 0.0, 1.0};
    bool alive = i < rows;
    if (alive) {
        fib_dir(i, rows, d64);
        alive = hemi ? (d64[0] * hx + d64[1] * hy + d64[2] * hz) > 0.0 : true;
    }
    const bool alive0 = alive;   // launched row (its hit list is written)
    float ox = (float)sx, oy = (float)sy, oz = (float)sz;
    float dx = (float)d64[0], dy = (float)d64[1], dz = (float)d64[2];
    int skip = -1;
    uint64_t acc = 0, acc1 = 0;
    int hid[KM];   // hit ids, stored after the walk (no store between the walk's loads)
#pragma unroll
    for (int q = 0; q < KM; ++q) hid[q] = -1;
    int* wst = stack + (BRUTE ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * RT_STACK4);
    for (int b = 0; b < K; ++b) {
        if (__ballot(alive) == 0ull) break;
        float tt;
        int id;
        if (alive) ++nseg;
        int slot;
        if (BRUTE)
            slot = alive ? closest_hit<true>(s, ox, oy, oz, dx, dy, dz, (float)RT_EPS, skip, nullptr, 0, tt, id) : -1;
        else if (CNT)
            slot = alive ? closest_hit<false, true>(s, ox, oy, oz, dx, dy, dz, (float)RT_EPS, skip,
                                                    stack + threadIdx.x, DISC_B, tt, id, &wc)
                         : -1;
        else
            slot = closest_hit_wave4(s, alive, ox, oy, oz, dx, dy, dz, (float)RT_EPS, skip, wst, tt, id);
        alive = alive && slot >= 0;
        if (alive) {
            const uint64_t field = (uint64_t)(__float_as_int(s.tri4[3 * slot + 1].w) + 1);
            if (W == 1 || b < 3)
                acc |= field << (RT_KEY_BITS * b);
            else
                acc1 |= field << (RT_KEY_BITS * (b - 3));
            // constant indices only, so the ids and keys stay in registers
#pragma unroll
            for (int q = 0; q < KM; ++q) {
                hid[q] = b == q ? id : hid[q];
                keys[q] = b == q ? acc : keys[q];
                if (W == 2) keys1[q] = b == q ? acc1 : keys1[q];
            }
            float px = ox + tt * dx, py = oy + tt * dy, pz = oz + tt * dz;
            reflect32(s.tri4[3 * slot + 1], s.tri4[3 * slot + 2], dx, dy, dz);
            ox = px;
            oy = py;
            oz = pz;
            skip = id;
        }
    }
    if (hits && alive0)
#pragma unroll
        for (int b = 0; b < KM; ++b)
            if (b < K) hits[i * K + b] = hid[b];
#pragma unroll
    for (int b = 0; b < KM; ++b) {
        const uint64_t left = __shfl_up(keys[b], 1, 64);
        const uint64_t left1 = W == 2 ? __shfl_up(keys1[b], 1, 64) : 0ull;
        const bool first = (threadIdx.x & 63) == 0 || left != keys[b] || (W == 2 && left1 != keys1[b]);
        if (b < K && keys[b] != 0ull && first) {
            if (W == 1)
                hash_insert(table, mask, max_probe, keys[b], overflow);
            else
                hash_insert2(table, mask, max_probe, keys[b], keys1[b], overflow);
        }
    }
    wave_count_add(segs, nseg);
    if (CNT) {
        wave_count_add(work + 0, wc.nodes);
        wave_count_add(work + 1, wc.tris);
        wave_count_add(work + 2, nseg);
    }
}

// Discovery with four lanes per ray (closest_hit_quad), for rays that are
// sparse against the triangles.  Otherwise as k_discover: the same rows, hits,
// keys and counts; a ray's key equal to that of the ray four lanes to the left
// is inserted there.  DQ_STK: stack entries per ray.
template <int STK, int KM>
__global__ __launch_bounds__(DISC_B) void k_discover_quad(SceneView s, double sx, double sy, double sz,
                                                          const int32_t* perm, const int32_t* off, int64_t rows,
                                                          int hemi, double hx, double hy, double hz, int K,
                                                          int32_t* hits, unsigned long long* segs,
                                                          unsigned long long* table, uint64_t mask,
                                                          uint64_t max_probe, int* overflow)
{
    constexpr int W = KM > RT_KM_SMALL ? 2 : 1;
    constexpr int DQ_STK = 3 * (STK / 2) + 4;   // a 4-wide node leaves at most three entries behind per two levels
    __shared__ int2 stack[DQ_STK * (DISC_B / 4)];
    const int64_t t = ((int64_t)blockIdx.x * DISC_B + threadIdx.x) >> 2;
    const int e = threadIdx.x & 3;
    unsigned nseg = 0;
    uint64_t keys[KM], keys1[KM];
#pragma unroll
    for (int q = 0; q < KM; ++q) keys[q] = keys1[q] = 0ull;
    const int64_t ch = t / RT_FIB_CHUNK;
    const int64_t i = ch * RT_FIB_CHUNK + perm[(off[ch] + (int)(t % RT_FIB_CHUNK)) % RT_FIB_CHUNK];
    double d64[3] = {0.0, 0.0, 1.0};
    bool alive = i < rows;
    if (alive) {
        fib_dir(i, rows, d64);
        alive = hemi ? (d64[0] * hx + d64[1] * hy + d64[2] * hz) > 0.0 : true;
    }
    const bool alive0 = alive;
    float ox = (float)sx, oy = (float)sy, oz = (float)sz;
    float dx = (float)d64[0], dy = (float)d64[1], dz = (float)d64[2];
    int skip = -1;
    uint64_t acc = 0, acc1 = 0;
    int hid[KM];
#pragma unroll
    for (int q = 0; q < KM; ++q) hid[q] = -1;
    int2* st = stack + (threadIdx.x >> 2);
    for (int b = 0; b < K; ++b) {
        if (__ballot(alive) == 0ull) break;
        float tt;
        int id;
        if (alive && e == 0) ++nseg;
        const int slot =
            closest_hit_quad(s, alive, ox, oy, oz, dx, dy, dz, (float)RT_EPS, skip, st, DISC_B / 4, tt, id);
        alive = alive && slot >= 0;
        if (alive) {
            const float4 tb = s.tri4[3 * (int64_t)slot + 1], tc = s.tri4[3 * (int64_t)slot + 2];
            const uint64_t field = (uint64_t)(__float_as_int(tb.w) + 1);
            if (W == 1 || b < 3)
                acc |= field << (RT_KEY_BITS * b);
            else
                acc1 |= field << (RT_KEY_BITS * (b - 3));
#pragma unroll
            for (int q = 0; q < KM; ++q) {
                hid[q] = b == q ? id : hid[q];
                keys[q] = b == q ? acc : keys[q];
                if (W == 2) keys1[q] = b == q ? acc1 : keys1[q];
            }
            const float px = ox + tt * dx, py = oy + tt * dy, pz = oz + tt * dz;
            reflect32(tb, tc, dx, dy, dz);
            ox = px;
            oy = py;
            oz = pz;
            skip = id;
        }
    }
    if (hits && alive0 && e == 0)
#pragma unroll
        for (int b = 0; b < KM; ++b)
            if (b < K) hits[i * K + b] = hid[b];
#pragma unroll
    for (int b = 0; b < KM; ++b) {
        const uint64_t left = __shfl_up(keys[b], 4, 64);
        const uint64_t left1 = W == 2 ? __shfl_up(keys1[b], 4, 64) : 0ull;
        const bool first = (threadIdx.x & 63) < 4 || left != keys[b] || (W == 2 && left1 != keys1[b]);
        if (b < K && e == 0 && keys[b] != 0ull && first) {
            if (W == 1)
                hash_insert(table, mask, max_probe, keys[b], overflow);
            else
                hash_insert2(table, mask, max_probe, keys[b], keys1[b], overflow);
        }
    }
    wave_count_add(segs, nseg);
}

// --------------------------------------------------------------------------
// 2. candidate keys: surface ids + 1, 21 bits per bounce; 0 = none
// --------------------------------------------------------------------------
// every sequence of <= K surfaces without immediate repeat, as keys of W
// words (0 for skipped)
template <int W>
__global__ void k_exhaustive_keys(int64_t n_surf, int K, int64_t total, uint64_t* keys)
{
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    // idx enumerates order k = 1..K blocks of n_surf^k entries
    int64_t base = 0, cnt = n_surf;
    int k = 1;
    while (k <= K && idx >= base + cnt) {
        base += cnt;
        cnt *= n_surf;
        ++k;
    }
    int64_t r = idx - base;
    uint64_t key = 0, key1 = 0;
    int prev = -1;
    bool ok = true;
    for (int j = 0; j < k; ++j) {
        int sidx = (int)(r % n_surf);
        r /= n_surf;
        if (sidx == prev) ok = false;
        prev = sidx;
        if (j < 3)
            key |= (uint64_t)(sidx + 1) << (RT_KEY_BITS * j);
        else
            key1 |= (uint64_t)(sidx + 1) << (RT_KEY_BITS * (j - 3));
    }
    keys[W * idx] = ok ? key : 0ull;
    if (W == 2) keys[W * idx + 1] = ok ? key1 : 0ull;
}

// surface id (or -1) of position j of a key of W words
template <int W>
__device__ __forceinline__ int key_surface(const uint64_t* key, int j)
{
    const uint64_t w = (W == 2 && j >= 3) ? key[1] : key[0];
    const int sh = RT_KEY_BITS * (j >= 3 ? j - 3 : j);
    const uint64_t v = (w >> sh) & ((1ull << RT_KEY_BITS) - 1);
    return v ? (int)v - 1 : -1;
}

// --------------------------------------------------------------------------
// 3. candidates: decode keys, images of the source
// --------------------------------------------------------------------------
// per candidate: order, KM surface ids (-1 padded), KM images (3 doubles each)
template <int KM>
__global__ void k_cand_prep(const uint64_t* keys, int64_t n, SceneView s, double sx, double sy, double sz,
                            int32_t* ck, int32_t* cseq, double* cimg)
{
    constexpr int W = KM > RT_KM_SMALL ? 2 : 1;
    int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    const uint64_t* key = keys + W * c;
    int k = 0;
    int seq[KM];
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        seq[j] = key_surface<W>(key, j);
        if (seq[j] >= 0 && k == j) k = j + 1;
    }
    ck[c] = k;
    double I[3] = {sx, sy, sz};
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        cseq[KM * c + j] = seq[j];
        if (j < k) {
            double o[3];
            mirror(s.s_plane + RT_PLANE * seq[j], I, o);
            I[0] = o[0];
            I[1] = o[1];
            I[2] = o[2];
        }
        cimg[3 * KM * c + 3 * j + 0] = I[0];
        cimg[3 * KM * c + 3 * j + 1] = I[1];
        cimg[3 * KM * c + 3 * j + 2] = I[2];
    }
}

// --------------------------------------------------------------------------
// 4. path geometry per (rx, candidate); valid cells compacted per wave
// --------------------------------------------------------------------------
struct CandView {
    const int32_t* k;
    const int32_t* seq;
    const double* img;
    int64_t n;
};

template <int KM>
__device__ __forceinline__ bool geo_path(const SceneView& s, const CandView& cv, int64_t c, const double* S,
                                         const double* X, double (*P)[3], int* tri, int& k)
{
    k = cv.k[c];
    int seq[KM];
    double I[KM + 1][3];
    I[0][0] = S[0];
    I[0][1] = S[1];
    I[0][2] = S[2];
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        seq[j] = cv.seq[KM * c + j];
        for (int q = 0; q < 3; ++q) I[j + 1][q] = cv.img[3 * KM * c + 3 * j + q];
    }
    return image_backtrace<KM>(s, seq, k, I, X, P, tri);
}



// occupied slots of the hash set, appended per wave (order is fixed by the sort that follows)
constexpr int TC_B = 256, TC_PT = 8;
// The occupied slots appended to out[1..] (out[0] = 0: the order-0 key).
__global__ __launch_bounds__(TC_B) void k_table_compact(const unsigned long long* table, int64_t cap, uint64_t* out,
                                                        int64_t out_cap, unsigned long long* counter)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) out[0] = 0ull;
    out += 1;
    __shared__ uint64_t vals[TC_B * TC_PT];
    __shared__ int n;
    __shared__ unsigned long long base;
    BlockAppend<TC_B * TC_PT> app{vals, &n, &base};
    app.init();
    unsigned long long v[TC_PT];   // all loads in flight before the first append
    for (int j = 0; j < TC_PT; ++j) {
        const int64_t i = ((int64_t)blockIdx.x * TC_PT + j) * TC_B + threadIdx.x;
        v[j] = i < cap ? table[i] : 0ull;
    }
    for (int j = 0; j < TC_PT; ++j)
        if (v[j] != 0ull) app.push((uint64_t)v[j]);
    app.flush(out, out_cap, counter);
}

// The same for two-word slots (word 1 loses its written bit): the block
// gathers slot indices, then copies both words.
__global__ __launch_bounds__(TC_B) void k_table_compact2(const unsigned long long* table, int64_t cap, uint64_t* out,
                                                         int64_t out_cap, unsigned long long* counter)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        out[0] = 0ull;
        out[1] = 0ull;
    }
    out += 2;
    __shared__ uint64_t idx[TC_B * TC_PT];
    __shared__ int n;
    __shared__ unsigned long long base;
    if (threadIdx.x == 0) n = 0;
    __syncthreads();
    for (int j = 0; j < TC_PT; ++j) {
        const int64_t i = ((int64_t)blockIdx.x * TC_PT + j) * TC_B + threadIdx.x;
        if (i < cap && table[2 * i] != 0ull) idx[atomicAdd(&n, 1)] = (uint64_t)i;
    }
    __syncthreads();
    const int cnt = n;
    if (threadIdx.x == 0) base = cnt > 0 ? atomicAdd(counter, (unsigned long long)cnt) : 0ull;
    __syncthreads();
    for (int t = threadIdx.x; t < cnt; t += TC_B) {
        const unsigned long long o = base + (unsigned long long)t;
        if (o < (unsigned long long)out_cap) {
            const uint64_t i = idx[t];
            out[2 * o] = table[2 * i];
            out[2 * o + 1] = table[2 * i + 1] & ~RT_W1_SET;
        }
    }
}

// Sort keys of the receivers: the Morton code of the position (up to 14 bits
// per axis over the scene's box, clamped to it) above the 22-bit index.  A
// scene without triangles has no box (null): every code is 0.  The order only
// groups the work, so it takes two bits per axis more than a square grid of R
// receivers has (24 bits for 64 x 64, three sort passes instead of six).
constexpr int RX_IDX_BITS = 22;
constexpr int64_t RX_SORT_MIN = 256;   // most receivers that go unsorted
static int rx_axis_bits(int64_t R)
{
    int lg = 0;
    while (((int64_t)1 << lg) < R) ++lg;
    return std::min(14, (lg + 1) / 2 + 2);
}
__global__ void k_rx_keys(const double* rx, int64_t R, const float* box, int bits, uint64_t* keys)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= R) return;
    const float cells = (float)(1 << bits);
    uint64_t code = 0;
    for (int k = 0; k < 3 && box; ++k) {
        const float lo = box[k], ext = box[3 + k] - box[k];
        float u = ext > 0.0f ? ((float)rx[3 * r + k] - lo) / ext : 0.5f;
        u = fminf(fmaxf(u, 0.0f), 1.0f);
        const unsigned q = (unsigned)fminf(u * cells, cells - 1.0f);
        for (int b = 0; b < bits; ++b) code |= (uint64_t)((q >> b) & 1u) << (3 * b + 2 - k);
    }
    keys[r] = code << RX_IDX_BITS | (uint64_t)r;
}

// One wave takes GEO_CPW candidates for 64 receivers, so the candidate's
// surfaces, planes and triangles are wave-uniform (scalar loads, no divergence
// in the loops over a surface's triangles).  The receivers of a wave are 64
// consecutive ones of `order` (the receivers sorted by Morton code of their
// positions; null: as they come): neighbours, so that a candidate tends to fail for all lanes of a
// wave at the same bounce.  A block covers 32 candidates = one 32-bit word of
// the receiver's row of the validity mask (mask[r * n_words + w], bit b =
// candidate 32 w + b).
// grid: x = word (group of 32 candidates), y = block of 64 slots of `order`
constexpr int GEO_B = 256, GEO_CPW = 8;
template <int KM>
__global__ __launch_bounds__(GEO_B) void k_geo_mask(SceneView s, CandView cv, double sx, double sy, double sz,
                                                    const double* rx, const uint64_t* order, int64_t R,
                                                    int64_t n_words, uint32_t* mask)
{
    static_assert(GEO_B / 64 * GEO_CPW == 32, "one mask word per block");
    __shared__ uint32_t part[GEO_B / 64][64];
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int64_t slot = (int64_t)blockIdx.y * 64 + lane;
    const int64_t r = slot >= R ? R : order ? (int64_t)(order[slot] & ((1ull << RX_IDX_BITS) - 1ull)) : slot;
    uint32_t bits = 0;
    if (r < R) {
        const double S[3] = {sx, sy, sz};
        const double X[3] = {rx[3 * r], rx[3 * r + 1], rx[3 * r + 2]};
        const int64_t c0 = (int64_t)blockIdx.x * 32 + wib * GEO_CPW;
        for (int j = 0; j < GEO_CPW; ++j) {
            const int64_t c = c0 + j;
            if (c >= cv.n) break;
            double P[KM][3];
            int tri[KM];
            int k;
            if (geo_path<KM>(s, cv, c, S, X, P, tri, k)) bits |= 1u << j;
        }
    }
    part[wib][lane] = bits << (GEO_CPW * wib);
    __syncthreads();
    if (wib == 0 && r < R)
        mask[r * n_words + blockIdx.x] = part[0][lane] | part[1][lane] | part[2][lane] | part[3][lane];
}

// valid cells per receiver (one wave per receiver; entry R is 0)
__global__ void k_cell_count(const uint32_t* mask, int64_t R, int64_t n_words, int64_t* cnt)
{
    const int64_t r = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (r > R) return;
    int64_t n = 0;
    if (r < R)
        for (int64_t w = lane; w < n_words; w += 64) n += __popc(mask[r * n_words + w]);
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
    if (lane == 0) cnt[r] = n;
}

// cells r * n_cand + c of the set bits, in (receiver, candidate) order, from
// the receivers' exclusive offsets (one wave per receiver)
__global__ void k_cell_emit(const uint32_t* mask, int64_t R, int64_t n_words, int64_t n_cand, const int64_t* rstart,
                            uint64_t* cells)
{
    const int64_t r = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (r >= R) return;
    int64_t base = rstart[r];
    for (int64_t w0 = 0; w0 < n_words; w0 += 64) {
        const int64_t w = w0 + lane;
        uint32_t m = w < n_words ? mask[r * n_words + w] : 0u;
        const int cnt = __popc(m);
        int incl = cnt;
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        int64_t pos = base + (incl - cnt);
        while (m) {
            const int b = __ffs((int)m) - 1;
            m &= m - 1u;
            cells[pos++] = (uint64_t)(r * n_cand + w * 32 + b);
        }
        base += __shfl(incl, 63, 64);
    }
}

// --------------------------------------------------------------------------
// 5/6. legs and field of each geometric path, in (receiver, candidate) order
// --------------------------------------------------------------------------
constexpr int LEG_B = 128;

template <int KM>
struct PathRec {
    int32_t rx, cand, k;
    int32_t tri[KM];
};

// Path points by value, constant indices only: V[0] = S, V[j] = P[j - 1] for
// j <= k, X from k + 1 on (so leg j runs from V[j] to V[j + 1]).
template <int KM>
__device__ __forceinline__ void path_points(const double* S, const double (*P)[3], const double* X, int k,
                                            double (*V)[3])
{
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        V[0][q] = S[q];
#pragma unroll
        for (int j = 1; j <= KM; ++j) V[j][q] = k >= j ? P[j - 1][q] : X[q];
        V[KM + 1][q] = X[q];
    }
}

// the point before X on the path (S for a direct path), by value
template <int KM>
__device__ __forceinline__ void last_point(const double* S, const double (*P)[3], int k, double* L)
{
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        double v = S[q];
#pragma unroll
        for (int j = 1; j <= KM; ++j) v = k == j ? P[j - 1][q] : v;
        L[q] = v;
    }
}

__device__ __forceinline__ double seg_len(const double* a, const double* b)
{
    double w0 = b[0] - a[0], w1 = b[1] - a[1], w2 = b[2] - a[2];
    return sqrt(w0 * w0 + w1 * w1 + w2 * w2);
}

// Reflection points of a cell whose geometry k_geo_mask accepted: the
// back-trace of image_backtrace without its tests (they have passed; the
// triangles are looked up for the paths whose legs are clear).
template <int KM>
__device__ __forceinline__ void cell_points(const SceneView& s, const int* seq, int k, const double* img,
                                            const double* X, double (*P)[3])
{
#pragma clang fp contract(off)
    double Q[3] = {X[0], X[1], X[2]};
#pragma unroll
    for (int i = KM; i >= 1; --i) {
        if (i > k) continue;
        const double* pl = s.s_plane + RT_PLANE * (int64_t)seq[i - 1];
        const double* I = img + 3 * (i - 1);
        const double w0 = Q[0] - I[0], w1 = Q[1] - I[1], w2 = Q[2] - I[2];
        const double den = pl[0] * w0 + pl[1] * w1 + pl[2] * w2;
        const double sp = div_fast(pl[3] - (pl[0] * I[0] + pl[1] * I[1] + pl[2] * I[2]), den);
        P[i - 1][0] = Q[0] = I[0] + sp * w0;
        P[i - 1][1] = Q[1] = I[1] + sp * w1;
        P[i - 1][2] = Q[2] = I[2] + sp * w2;
    }
}

template <bool BRUTE, bool FIELD, int STK, int KM>
__global__ __launch_bounds__(LEG_B) void k_paths(SceneView s, CandView cv, TraceConst tc, double sx, double sy,
                                                 double sz, const double* rx, const uint64_t* cells, int64_t n,
                                                 uint8_t* valid, float2* amp, double* len, PathRec<KM>* recs,
                                                 unsigned long long* segs, unsigned long long* n_valid)
{
    __shared__ int stack[STK * LEG_B];
    int64_t i = (int64_t)blockIdx.x * LEG_B + threadIdx.x;
    unsigned nseg = 0, nval = 0;
    if (i < n) {
        const uint64_t cell = cells[i];
        const int64_t r = (int64_t)(cell / (uint64_t)cv.n), c = (int64_t)(cell - (uint64_t)r * cv.n);
        double S[3] = {sx, sy, sz};
        double X[3] = {rx[3 * r], rx[3 * r + 1], rx[3 * r + 2]};
        double P[KM][3];
        int tri[KM];
#pragma unroll
        for (int j = 0; j < KM; ++j) tri[j] = -1;
        int sq[KM];
#pragma unroll
        for (int j = 0; j < KM; ++j) sq[j] = cv.seq[KM * c + j];
        const int k = cv.k[c];
        cell_points<KM>(s, sq, k, cv.img + 3 * KM * c, X, P);
        bool ok = true;
        float Ft = 1.0f, Fr = 1.0f;
        double V[KM + 2][3];
        path_points<KM>(S, P, X, k, V);
        if (FIELD && ok) {
            double v1[3], vl[3], L[3];
            last_point<KM>(S, P, k, L);
            for (int q = 0; q < 3; ++q) {
                v1[q] = V[1][q] - S[q];
                vl[q] = L[q] - X[q];
            }
            const bool on_t = pattern_gate_amp(tc.txa.pattern, tc.txa.param, v1, tc.txa.axis, tc.txa.axis_norm, Ft);
            const bool on_r = pattern_gate_amp(tc.rxa.pattern, tc.rxa.param, vl, tc.rxa.axis, tc.rxa.axis_norm, Fr);
            ok = on_t && on_r;
        }
#pragma unroll
        for (int j = 0; j <= KM; ++j) {
            if (j > k || !ok) break;
            // leg j runs from V[j] to V[j + 1] (V[j + 1] = X when j = k)
            const int sa = j == 0 ? -1 : sq[j > 0 ? j - 1 : 0];
            const int sb = j == k ? -1 : sq[j < KM ? j : 0];
            ++nseg;
            if (leg_blocked<BRUTE>(s, V[j], V[j + 1], sa, sb, stack + threadIdx.x, LEG_B)) ok = false;
        }
        if (ok)
#pragma unroll
            for (int j = 0; j < KM; ++j)
                if (j < k) tri[j] = surface_contains(s, sq[j], P[j]);
        valid[i] = ok ? 1 : 0;
        nval = ok ? 1 : 0;
        PathRec<KM> pr;
        pr.rx = (int32_t)r;
        pr.cand = (int32_t)c;
        pr.k = k;
#pragma unroll
        for (int j = 0; j < KM; ++j) pr.tri[j] = j < k ? tri[j] : -1;
        recs[i] = pr;
        if (FIELD) {
            double D = 0.0, Lj[KM + 1];
#pragma unroll
            for (int j = 0; j <= KM; ++j) {
                Lj[j] = 0.0;
                if (j <= k) {
                    Lj[j] = seg_len(V[j], V[j + 1]);
                    D += Lj[j];
                }
            }
            float2 a = make_float2(0.0f, 0.0f);
            if (ok) {
                float ar = 1.0f, ai = 0.0f;
#pragma unroll
                for (int j = 0; j < KM; ++j) {
                    if (j >= k) break;
                    float2 Rc;
                    if (tc.fresnel) {
                        const double d[3] = {V[j + 1][0] - V[j][0], V[j + 1][1] - V[j][1], V[j + 1][2] - V[j][2]};
                        Rc = fresnel_coef(s, tri[j], d, Lj[j], tc.fresnel, tc.sig_scale);
                    } else {
                        Rc = s.refl[tri[j]];
                    }
                    float nr = ar * Rc.x - ai * Rc.y;
                    float ni = ar * Rc.y + ai * Rc.x;
                    ar = nr;
                    ai = ni;
                }
                float mag = sqrtf((float)tc.two_eta0_pt_gt) * Ft * sqrtf((float)tc.rxa.gain) * Fr *
                            (tc.lam_4pi * __builtin_amdgcn_rcpf((float)D));
                float cs, sn;
                phase_cs(D, tc.inv_lambda, cs, sn);
                a = make_float2(mag * (ar * cs - ai * sn), mag * (ar * sn + ai * cs));
            }
            amp[i] = a;
            len[i] = D;
        }
    }
    wave_count_add(segs, nseg);
    if (FIELD) wave_count_add(n_valid, nval);
}

// E_env[r] = sum of emitted paths of receiver r (FP64): one wave per
// receiver, lane l sums records l, l + 64, ... of its range, then a fixed
// butterfly over the lanes (the same order on every run).
constexpr int ENV_B = 256;
__global__ __launch_bounds__(ENV_B) void k_env_reduce(const int64_t* rstart, int64_t R, const uint8_t* valid,
                                                      const float2* amp, float2* E)
{
    const int64_t r = (int64_t)blockIdx.x * (ENV_B / 64) + (threadIdx.x >> 6);
    if (r >= R) return;   // whole waves leave together
    const int lane = threadIdx.x & 63;
    double er = 0.0, ei = 0.0;
    const int64_t j1 = rstart[r + 1];
    for (int64_t j = rstart[r] + lane; j < j1; j += 64)
        if (valid[j]) {
            const float2 a = amp[j];
            er += (double)a.x;
            ei += (double)a.y;
        }
    for (int o = 32; o > 0; o >>= 1) {
        er += __shfl_xor(er, o, 64);
        ei += __shfl_xor(ei, o, 64);
    }
    if (lane == 0) E[r] = make_float2((float)er, (float)ei);
}

// keep valid records: env path records for read-back
template <int KM>
__global__ void k_env_compact(const PathRec<KM>* recs, CandView cv, const uint8_t* valid, const int64_t* off2,
                              const float2* amp, const double* len, int64_t n, EnvRec* out)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || !valid[i]) return;
    const PathRec<KM>& pr = recs[i];
    EnvRec e;
    e.rx = pr.rx;
    e.order = pr.k;
#pragma unroll
    for (int j = 0; j < RT_MAX_K; ++j) {
        e.seq[j] = -1;
        e.tri[j] = -1;
    }
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        e.seq[j] = cv.seq[KM * pr.cand + j];
        e.tri[j] = pr.tri[j];
    }
    e.length = len[i];
    e.amp[0] = amp[i].x;
    e.amp[1] = amp[i].y;
    out[off2[i]] = e;
}

// Rows of useq_stride(KM) = 2 KM + 2 ints: rx, surfaces s_0..s_{KM-1},
// triangles t_0..t_{KM-1} reached from the centre, 0.
constexpr int useq_stride(int KM) { return 2 * KM + 2; }

// The centre branch's valid sequences of order >= 1, by receiver (one wave
// each, its records in candidate order): their number (entry R is 0), and the
// receiver's place in the launch order of the per-element kernel, heaviest
// first (the longest waves start first and short ones fill the tail): key =
// inverted cost (slots weighted by legs, 20 bits) above the receiver index.
// Bound by launches (4-8 us each, a read of 24 bytes a record): by receiver it
// is this, a scan of R + 1 counts and k_u_emit, where flags, their scan, the
// rows, the pointers and the order from the rows were seven launches; with the
// receivers' order off the Tx stream a map of 61 x 91 receivers in 1 cm steps went from 720 to
// 554 us, a box of 12 triangles from 411 to 356.
template <int KM>
__global__ void k_u_count(const int64_t* rstart, const PathRec<KM>* recs, const uint8_t* valid, int64_t R,
                          int64_t* cnt, uint64_t* keys)
{
    const int64_t r = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (r > R) return;
    int n = 0, legs = 0;
    if (r < R)
        for (int64_t i = rstart[r] + lane; i < rstart[r + 1]; i += 64)
            if (valid[i] && recs[i].k >= 1) {
                ++n;
                legs += recs[i].k + 1;
            }
    for (int o = 32; o > 0; o >>= 1) {
        n += __shfl_xor(n, o, 64);
        legs += __shfl_xor(legs, o, 64);
    }
    if (lane != 0) return;
    cnt[r] = n;
    if (r < R) {
        const uint64_t cost = 1 + (uint64_t)legs;   // the direct slot: one leg
        keys[r] = ((0xFFFFFull - (cost < 0xFFFFFull ? cost : 0xFFFFFull)) << 32) | (uint64_t)r;
    }
}

// their rows, receiver r's from uptr[r] on
template <int KM>
__global__ void k_u_emit(const int64_t* rstart, const PathRec<KM>* recs, CandView cv, const uint8_t* valid, int64_t R,
                         const int64_t* uptr, int32_t* useq)
{
    constexpr int US = useq_stride(KM);
    const int64_t r = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (r >= R) return;
    int64_t o = uptr[r];
    const int64_t e = rstart[r + 1];
    for (int64_t i0 = rstart[r]; i0 < e; i0 += 64) {
        const int64_t i = i0 + lane;
        const bool take = i < e && valid[i] && recs[i].k >= 1;
        const unsigned long long m = __ballot(take);
        if (take) {
            int32_t* row = useq + US * (o + __popcll(m & ((1ull << lane) - 1ull)));
            row[0] = (int32_t)r;
#pragma unroll
            for (int j = 0; j < KM; ++j) {
                row[1 + j] = cv.seq[KM * (int64_t)recs[i].cand + j];
                row[1 + KM + j] = recs[i].tri[j];
            }
            row[US - 1] = 0;
        }
        o += __popcll(m);
    }
}

// --------------------------------------------------------------------------
// 7. RIS
// --------------------------------------------------------------------------
// Field reaching element m (eqs. (4)-(6) without Gamma_m and F_out):
// T = sum over incoming paths p of A_t(v1_p) sqrt(G F_in(p) d_y d_z / 4pi)
// prod(R_p) e^{-jk d_p} / d_p; the direct leg, plus the reflections Tx ->
// surfaces -> m when they are modelled.
struct TxmRec {
    float2 T;
    int ok;        // some incoming path emitted (clear legs, F_t, F_in > 0)
    int pad;
};

template <bool BRUTE, int STK>
__global__ __launch_bounds__(64) void k_txm(SceneView s, TraceConst tc, RisView rv, TxmRec* out,
                                            unsigned long long* segs)
{
    __shared__ int stack[STK * 64];
    int m = blockIdx.x * 64 + threadIdx.x;
    unsigned nseg = 0;
    if (m < rv.M) {
        const double* e = rv.elem + 3 * m;
        double vt[3] = {e[0] - tc.tx[0], e[1] - tc.tx[1], e[2] - tc.tx[2]};
        double back[3] = {-vt[0], -vt[1], -vt[2]};
        double dt = sqrt(vt[0] * vt[0] + vt[1] * vt[1] + vt[2] * vt[2]);
        const double ct = cos_between(vt, tc.txa.axis, tc.txa.axis_norm);
        const double ci = cos_between(back, rv.normal, rv.normal_norm);
        const float Ft = pattern_amp(tc.txa.pattern, tc.txa.param, ct);   // sqrt(F_t)
        const float Fin = pattern_amp(1, rv.q, ci);                        // sqrt(F_in)
        bool ok = pattern_on(tc.txa.pattern, ct) && pattern_on(1, ci);
        if (ok) {
            ++nseg;
            ok = !leg_blocked<BRUTE>(s, tc.tx, e, -1, -1, stack + threadIdx.x, 64);
        }
        TxmRec r;
        r.ok = ok ? 1 : 0;
        r.pad = 0;
        r.T = make_float2(0.0f, 0.0f);
        if (ok) {
            const float fac = (float)(sqrt(tc.two_eta0_pt_gt) * (double)Ft *
                                      sqrt(rv.gain * rv.dy * rv.dz / (4.0 * 3.141592653589793)) * (double)Fin / dt);
            float cs, sn;
            phase_cs(dt, tc.inv_lambda, cs, sn);
            r.T = make_float2(fac * cs, fac * sn);
        }
        out[m] = r;
    }
    wave_count_add(segs, nseg);
}

// Incoming reflections (Section II-B, supporting reflections): the image
// method from the Tx to the RIS, restricted like the out side to the
// sequences valid from the Tx to the RIS centre u.
// 1) per Tx candidate of order >= 1: valid and unblocked from the Tx to u?
template <bool BRUTE, int STK, int KM>
__global__ __launch_bounds__(LEG_B) void k_in_centre(SceneView s, CandView cv, double sx, double sy, double sz,
                                                     double ux, double uy, double uz, uint8_t* ok_out,
                                                     unsigned long long* segs)
{
    __shared__ int stack[STK * LEG_B];
    const int64_t c = (int64_t)blockIdx.x * LEG_B + threadIdx.x;
    unsigned nseg = 0;
    if (c < cv.n) {
        const double S[3] = {sx, sy, sz};
        const double X[3] = {ux, uy, uz};
        double P[KM][3];
        int tri[KM];
        int k = 0;
        bool ok = cv.k[c] >= 1 && geo_path<KM>(s, cv, c, S, X, P, tri, k);
        double V[KM + 2][3];
        path_points<KM>(S, P, X, k, V);
        int sq[KM];
#pragma unroll
        for (int j = 0; j < KM; ++j) sq[j] = cv.seq[KM * c + j];
#pragma unroll
        for (int j = 0; j <= KM; ++j) {
            if (j > k || !ok) break;
            const int sa = j == 0 ? -1 : sq[j > 0 ? j - 1 : 0];
            const int sb = j == k ? -1 : sq[j < KM ? j : 0];
            ++nseg;
            if (leg_blocked<BRUTE>(s, V[j], V[j + 1], sa, sb, stack + threadIdx.x, LEG_B)) ok = false;
        }
        ok_out[c] = ok ? 1 : 0;
    }
    wave_count_add(segs, nseg);
}

__global__ void k_in_list(const uint8_t* ok, const int64_t* off, int64_t n, int32_t* list)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c < n && ok[c]) list[off[c]] = (int32_t)c;
}

// 2) per (sequence j of the list, element m): the path Tx -> seq -> m, its legs
// and its contribution to T_m (zero if not emitted); *n_in = list length
template <bool BRUTE, int STK, int KM>
__global__ __launch_bounds__(LEG_B) void k_in_elem(SceneView s, CandView cv, TraceConst tc, RisView rv,
                                                   const int32_t* list, const int64_t* n_in, float2* contrib,
                                                   uint8_t* emitted_out, unsigned long long* segs,
                                                   unsigned long long* n_paths)
{
    __shared__ int stack[STK * LEG_B];
    const int64_t i = (int64_t)blockIdx.x * LEG_B + threadIdx.x;
    const int64_t M = rv.M;
    const int64_t nl = *n_in;
    unsigned nseg = 0, emitted = 0;
    if (i < nl * M) {
        const int64_t j = i / M, m = i - j * M;
        const int64_t c = list[j];
        const double S[3] = {tc.tx[0], tc.tx[1], tc.tx[2]};
        const double X[3] = {rv.elem[3 * m], rv.elem[3 * m + 1], rv.elem[3 * m + 2]};
        double P[KM][3];
        int tri[KM];
        int k = 0;
        bool ok = geo_path<KM>(s, cv, c, S, X, P, tri, k);
        double V[KM + 2][3];
        path_points<KM>(S, P, X, k, V);
        float Ft = 0.0f, Fin = 0.0f;
        if (ok) {
            double v1[3], back[3], L[3];
            last_point<KM>(S, P, k, L);
            for (int q = 0; q < 3; ++q) {
                v1[q] = V[1][q] - S[q];
                back[q] = L[q] - X[q];
            }
            const double ct = cos_between(v1, tc.txa.axis, tc.txa.axis_norm);
            const double ci = cos_between(back, rv.normal, rv.normal_norm);
            Ft = pattern_amp(tc.txa.pattern, tc.txa.param, ct);
            Fin = pattern_amp(1, rv.q, ci);
            ok = pattern_on(tc.txa.pattern, ct) && pattern_on(1, ci);
        }
        int sq[KM];
#pragma unroll
        for (int q = 0; q < KM; ++q) sq[q] = cv.seq[KM * c + q];
#pragma unroll
        for (int q = 0; q <= KM; ++q) {
            if (q > k || !ok) break;
            const int sa = q == 0 ? -1 : sq[q > 0 ? q - 1 : 0];
            const int sb = q == k ? -1 : sq[q < KM ? q : 0];
            ++nseg;
            if (leg_blocked<BRUTE>(s, V[q], V[q + 1], sa, sb, stack + threadIdx.x, LEG_B)) ok = false;
        }
        float2 a = make_float2(0.0f, 0.0f);
        if (ok) {
            double D = 0.0, Lq[KM + 1];
#pragma unroll
            for (int q = 0; q <= KM; ++q) {
                Lq[q] = 0.0;
                if (q <= k) {
                    Lq[q] = seg_len(V[q], V[q + 1]);
                    D += Lq[q];
                }
            }
            float ar = 1.0f, ai = 0.0f;
#pragma unroll
            for (int q = 0; q < KM; ++q) {
                if (q >= k) break;
                float2 Rc;
                if (tc.fresnel) {
                    const double d[3] = {V[q + 1][0] - V[q][0], V[q + 1][1] - V[q][1], V[q + 1][2] - V[q][2]};
                    Rc = fresnel_coef(s, tri[q], d, Lq[q], tc.fresnel, tc.sig_scale);
                } else {
                    Rc = s.refl[tri[q]];
                }
                const float nr = ar * Rc.x - ai * Rc.y;
                const float ni = ar * Rc.y + ai * Rc.x;
                ar = nr;
                ai = ni;
            }
            const float mag = (float)(sqrt(tc.two_eta0_pt_gt) * (double)Ft *
                                      sqrt(rv.gain * rv.dy * rv.dz / (4.0 * 3.141592653589793)) * (double)Fin / D);
            float cs, sn;
            phase_cs(D, tc.inv_lambda, cs, sn);
            a = make_float2(mag * (ar * cs - ai * sn), mag * (ar * sn + ai * cs));
            emitted = 1;
        }
        contrib[i] = a;
        emitted_out[i] = (uint8_t)emitted;
    }
    wave_count_add(segs, nseg);
    wave_count_add(n_paths, emitted);
}

// 3) per element: T_m += the contributions of the list in list order (FP64)
__global__ void k_in_sum(const float2* contrib, const uint8_t* emitted, const int64_t* n_in, int64_t M,
                         TxmRec* txm)
{
    const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= M) return;
    const int64_t nl = *n_in;
    TxmRec r = txm[m];
    double tr = r.T.x, ti = r.T.y;
    bool lit = r.ok != 0;
    for (int64_t j = 0; j < nl; ++j) {
        const float2 a = contrib[j * M + m];
        if (emitted[j * M + m]) lit = true;
        tr += (double)a.x;
        ti += (double)a.y;
    }
    r.T = make_float2((float)tr, (float)ti);
    r.ok = lit ? 1 : 0;
    txm[m] = r;
}

constexpr int RIS_B = 128;

// Back-trace like image_backtrace, but each reflection first tries the
// triangle the RIS-centre path used (hint); a point on a surface lies in
// exactly one of its triangles, so the result is the same as a full search.
// S: the source; img: this lane's images 1 .. KM - 1 in LDS, [3][64] each;
// last: image k (used for k = KM).
typedef double lds_double __attribute__((may_alias));
template <bool CNT, int KM>
__device__ inline bool image_backtrace_hint(const SceneView& s, const int* seq, const int* hint, int k,
                                            const double* S, const lds_double* img, const double* last,
                                            const double* X, double (*P)[3], int* tri, WorkCount* wc)
{
#pragma clang fp contract(off)
    double Q[3] = {X[0], X[1], X[2]};
#pragma unroll
    for (int i = KM; i >= 1; --i) {
        if (i > k) continue;
        const double* pl = s.s_plane + RT_PLANE * seq[i - 1];
        double Im[3];
        for (int q = 0; q < 3; ++q) Im[q] = i == KM ? last[q] : img[(3 * (i - 1) + q) * 64];
        double w0 = Q[0] - Im[0], w1 = Q[1] - Im[1], w2 = Q[2] - Im[2];
        double den = pl[0] * w0 + pl[1] * w1 + pl[2] * w2;
        if (den == 0.0) return false;
        double sp = div_fast(pl[3] - (pl[0] * Im[0] + pl[1] * Im[1] + pl[2] * Im[2]), den);
        if (!(sp > 0.0 && sp < 1.0)) return false;
        double p[3] = {Im[0] + sp * w0, Im[1] + sp * w1, Im[2] + sp * w2};
        int h = hint[i - 1];
        if (CNT && h >= 0) wc->contain++;
        int t = (h >= 0 && contains_proj<true>(s, h, p)) ? h : surface_contains<CNT>(s, seq[i - 1], p, wc);
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
            prev[q] = i == 0 ? S[q] : P[i > 0 ? i - 1 : 0][q];
            next[q] = (i == k - 1 || i + 1 >= KM) ? X[q] : P[i + 1 < KM ? i + 1 : 0][q];
        }
        double a = plane_side(pl, prev);
        double b = plane_side(pl, next);
        if (!((a > 0.0 && b > 0.0) || (a < 0.0 && b < 0.0))) return false;
    }
    return true;
}

// CNT: counting build; work[0..4] += node visits, triangle tests,
// containment tests, (slot, element) pairs, legs.
//
// Waves a SIMD: bound by issue and latency together, so every wave more counts
// (lab room 1110 us with three, 945 with four; office floor 42 ms with two, 31
// with three).  Registers and LDS are cut to five for up to order 3 (96
// registers: lab room 880 us, 64 x 64 receivers among 50000 triangles 1030 ->
// 930) and to four above (28 ms): the images of the elements wait in the legs'
// LDS until the legs are written there, one or two legs stay in registers.  At
// 96 registers six are spilled (28 bytes of scratch a lane; 16 and 68 bytes with
// Fresnel coefficients): their traffic is less than the fifth wave hides.  The
// instances with more to keep stay at four.

// FRES: Fresnel coefficients of the materials (tc.fresnel) instead of the fixed ones
template <bool BRUTE, bool KEEP, int STK, bool CNT, bool FRES, int KM>
__global__ __launch_bounds__(RIS_B, KEEP || BRUTE || CNT || KM > RT_KM_SMALL ? 4 : 5) void k_ris(SceneView s, TraceConst tc, RisView rv, const TxmRec* txm,
                                               const double* rx, int64_t R, const int64_t* uptr,
                                               const int32_t* useq, const uint64_t* order, int n_mchunk, float2* H,
                                               uint8_t* rvalid, float2* camp, double* clen, unsigned long long* segs,
                                               unsigned long long* work, unsigned long long* fallbacks)
{
    // the rays of a slot's legs wait in LDS while earlier legs are walked (fewer live registers)
    static_assert(LegRays<KM>::LDS_FLOATS >= 6 * (KM - 1) * 64, "the images of a lane");
    __shared__ __attribute__((aligned(16))) float legbuf[RIS_B / 64][LegRays<KM>::LDS_FLOATS];
    // per-wave frontier and candidate lists of the tube walk; the frontier's room is the stack of the walks
    // leg by leg
    __shared__ int tfront[RIS_B / 64][2 * RT_TUBE_FRONT];
    __shared__ int tcand[RIS_B / 64][RT_TUBE_CAND];
    __shared__ float4 ttube[RIS_B / 64][3 * (KM + 1)];
    constexpr int US = useq_stride(KM);
    static_assert(2 * RT_TUBE_FRONT >= STK, "wave stack");
    WorkCount wc;
    unsigned pairs = 0;
    const int wib = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // wave in block (uniform)
    const int64_t w = (int64_t)blockIdx.x * (RIS_B / 64) + wib;
    const int lane = threadIdx.x & 63;
    int* my_stack = tfront[wib];
    LegRays<KM> legs;
    legs.lds = &legbuf[wib][lane];
    unsigned nseg = 0;
    unsigned n_fallback = 0;   // slots whose grouped leg walk fell back (wave-uniform)
    if (w < R * n_mchunk) {
        const int64_t wr = w / n_mchunk;
        const int64_t r = (int64_t)(order[wr] & 0xFFFFFFFFull);
        // the wave's 64 elements are neighbours on the RIS (Morton order of their
        // in-plane coordinates), so the legs of a slot stay in a thin tube
        const int mi = (int)(w - wr * n_mchunk) * 64 + lane;
        const bool active = mi < rv.M;
        const int mm = active ? rv.order[mi] : 0;
        const int m = mm;
        const double* e = rv.elem + 3 * mm;
        const double E[3] = {e[0], e[1], e[2]};
        double dt_keep = 0.0;   // |E - Tx| as the direct leg's length (kept paths only; 0 with the
                                // incoming reflections, whose element field sums several paths)
        if (KEEP && !(tc.flags & 32)) {
#pragma clang fp contract(off)
            const double v0 = E[0] - tc.tx[0], v1 = E[1] - tc.tx[1], v2 = E[2] - tc.tx[2];
            dt_keep = sqrt(v0 * v0 + v1 * v1 + v2 * v2);
        }
        const TxmRec t = txm[mm];
        const double X[3] = {rx[3 * r], rx[3 * r + 1], rx[3 * r + 2]};
        const int64_t u0 = uptr[r], u1 = uptr[r + 1];
        const int64_t nsl = 1 + (u1 - u0);
        double acc_r = 0.0, acc_i = 0.0;
#pragma unroll 1
        for (int64_t sl = 0; sl < nsl; ++sl) {
            // the slot's sequence is the same for every lane of the wave
            int seq[KM], hint[KM];
#pragma unroll
            for (int j = 0; j < KM; ++j) seq[j] = hint[j] = -1;
            int k = 0;
            if (sl > 0) {
                const int32_t* row = useq + US * (u0 + sl - 1);
#pragma unroll
                for (int j = 0; j < KM; ++j) {
                    seq[j] = row[1 + j];
                    hint[j] = row[1 + KM + j];
                    if (seq[j] >= 0) k = j + 1;
                }
            }
            bool ok = active && t.ok;
            if (CNT && active) ++pairs;
            // phase 1 (FP64): image method, leg rays, length, amplitude
            float amp_r = 0.0f, amp_i = 0.0f;
            double Dr_keep = 0.0;
            {
                double P[KM][3];
                int tri[KM];
#pragma unroll
                for (int j = 0; j < KM; ++j) tri[j] = -1;
                {
                    // The images wait in the room of the legs (KM = 5: 36 registers less), under other lanes' legs: a
                    // lane's reads stay ahead of its later writes (the two may alias), and the LDS operations of a
                    // wave keep their order.  (A fence here costs 6 to 18 % of a trace.)
                    lds_double* img = (lds_double*)&legbuf[wib][0] + lane;
                    double cur[3] = {E[0], E[1], E[2]};
#pragma unroll
                    for (int j = 0; j < KM; ++j)
                        if (j < k) {
                            double nx[3];
                            mirror(s.s_plane + RT_PLANE * seq[j], cur, nx);
                            for (int q = 0; q < 3; ++q) {
                                cur[q] = nx[q];
                                if (j + 1 < KM) img[(3 * j + q) * 64] = nx[q];
                            }
                        }
                    if (ok) ok = image_backtrace_hint<CNT, KM>(s, seq, hint, k, E, img, cur, X, P, tri, &wc);
                }
                float Fout = 0.0f, Fr = 0.0f;
                if (ok) {
                    // first and last path points, selected by value (constant indices)
                    double f[3], l[3];
                    last_point<KM>(E, P, k, l);
                    for (int q = 0; q < 3; ++q) f[q] = k ? P[0][q] : X[q];
                    double v1[3] = {f[0] - E[0], f[1] - E[1], f[2] - E[2]};
                    double vl[3] = {l[0] - X[0], l[1] - X[1], l[2] - X[2]};
                    const bool on_o = pattern_gate_amp(1, rv.q, v1, rv.normal, rv.normal_norm, Fout);   // sqrt(F_out)
                    const bool on_r =
                        pattern_gate_amp(tc.rxa.pattern, tc.rxa.param, vl, tc.rxa.axis, tc.rxa.axis_norm, Fr);   // sqrt(F_r)
                    ok = on_o && on_r;
                }
                double Dr = 0.0;
                double Lk[KM + 1];   // leg lengths (the Fresnel angles use them)
#pragma unroll
                for (int j = 0; j <= KM; ++j) {
                    Lk[j] = 0.0;
                    if (j <= k) {
#pragma clang fp contract(off)
                        const double* A = j == 0 ? E : P[j - 1];
                        const double* B = j == k ? X : P[j];
                        double w0 = B[0] - A[0], w1 = B[1] - A[1], w2 = B[2] - A[2];
                        double L, il;   // the leg ray's direction as leg_blocked forms it
                        sqrt_inv(w0 * w0 + w1 * w1 + w2 * w2, L, il);
                        if (FRES) Lk[j] = L;
                        Dr += L;
                        legs.set(j, 0, (float)A[0]);
                        legs.set(j, 1, (float)A[1]);
                        legs.set(j, 2, (float)A[2]);
                        legs.set(j, 3, (float)(w0 * il));
                        legs.set(j, 4, (float)(w1 * il));
                        legs.set(j, 5, (float)(w2 * il));
                        legs.set(j, 6, (float)(L - RT_EPS));
                    }
                }
                if (KEEP) Dr_keep = Dr;
                if (ok) {
                    float ar = 1.0f, ai = 0.0f;
#pragma unroll
                    for (int j = 0; j < KM; ++j) {
                        if (j >= k) break;
                        float2 Rc;
                        if (FRES) {
                            double d[3];
                            for (int q = 0; q < 3; ++q) d[q] = P[j][q] - (j == 0 ? E[q] : P[j > 0 ? j - 1 : 0][q]);
                            Rc = fresnel_coef(s, tri[j], d, Lk[j], tc.fresnel, tc.sig_scale);
                        } else {
                            Rc = s.refl[tri[j]];
                        }
                        float nr = ar * Rc.x - ai * Rc.y;
                        float ni = ar * Rc.y + ai * Rc.x;
                        ar = nr;
                        ai = ni;
                    }
                    const float mag = Fout * sqrtf((float)tc.rxa.gain) * Fr * (tc.lam_4pi * __builtin_amdgcn_rcpf((float)Dr));
                    float cs, sn;
                    phase_cs(Dr, tc.inv_lambda, cs, sn);
                    // incoming field x reflections x out-going phase
                    const float zr = t.T.x * ar - t.T.y * ai, zi = t.T.x * ai + t.T.y * ar;
                    amp_r = mag * (zr * cs - zi * sn);
                    amp_i = mag * (zr * sn + zi * cs);
                }
            }
            // phase 2 (FP32): visibility of every leg, the wave walking the BVH together
            const float tmin = (float)RT_EPS;
            if (BRUTE || CNT) {
#pragma unroll 1
                for (int j = 0; j <= k; ++j) {
                    const int sa = leg_surface_a<KM>(seq, j);
                    const int sb = leg_surface_b<KM>(seq, j, k);
                    float ray[7];
                    legs.get(j, ray);
                    const float ox = ray[0], oy = ray[1], oz = ray[2], dx = ray[3], dy = ray[4], dz = ray[5];
                    const float tmax = ray[6];
                    if (ok) ++nseg;
                    const bool searching = ok && tmax > tmin;
                    bool blocked;
                    if (BRUTE)
                        blocked = searching &&
                                  any_hit<true>(s, ox, oy, oz, dx, dy, dz, tmin, tmax, sa, sb, nullptr, 0);
                    else   // the counting build walks the binary tree: its work is what is counted
                        blocked = any_hit_wave<true>(s, searching, ox, oy, oz, dx, dy, dz, tmin, tmax, sa, sb,
                                                     my_stack, &wc);
                    ok = ok && !blocked;
                }
            } else {
                // every leg at once; legs are counted as the sequential test would (up to the first blocked one)
                const float end[3] = {(float)X[0], (float)X[1], (float)X[2]};
                const unsigned res = legs_blocked_tube<KM>(s, ok, k, seq, legs, end, ttube[wib], tfront[wib],
                                                       tcand[wib]);
                n_fallback += (res & RT_TUBE_FELL_BACK) ? 1u : 0u;   // same on every lane
                const unsigned bl = res & ~RT_TUBE_FELL_BACK;
                if (ok) nseg += bl ? (unsigned)(__ffs((int)bl)) : (unsigned)(k + 1);
                ok = ok && bl == 0u;
            }
            if (ok) {
                acc_r += (double)amp_r;
                acc_i += (double)amp_i;
            }
            if (KEEP && active) {
                const int64_t cell = (u0 + r + sl) * rv.M + m;
                if (rvalid) rvalid[cell] = ok ? 1 : 0;
                if (camp) {   // per-path amplitude and unfolded length (d_t + D_r; D_r alone with the incoming
                              // reflections): impulse response and per-path read-back
                    camp[cell] = ok ? make_float2(amp_r, amp_i) : make_float2(0.0f, 0.0f);
                    clen[cell] = dt_keep + Dr_keep;
                }
            }
        }
        if (active) H[r * rv.M + m] = make_float2((float)acc_r, (float)acc_i);
    }
    if (CNT) {
        wave_count_add(work + 0, wc.nodes);
        wave_count_add(work + 1, wc.tris);
        wave_count_add(work + 2, wc.contain);
        wave_count_add(work + 3, pairs);
        wave_count_add(work + 4, nseg);
    }
    wave_count_add(segs, nseg);
    if (!BRUTE && !CNT) wave_count_add(fallbacks, lane == 0 ? n_fallback : 0u);
}

// --------------------------------------------------------------------------
// host orchestration
// --------------------------------------------------------------------------
#define SEL_BOOL(b, NAME, ...)            \
    if (b) {                              \
        constexpr bool NAME = true;       \
        __VA_ARGS__;                      \
    } else {                              \
        constexpr bool NAME = false;      \
        __VA_ARGS__;                      \
    }
#define SEL_STK(stk, ...)                 \
    if ((stk) == 32) {                    \
        constexpr int STK = 32;           \
        __VA_ARGS__;                      \
    } else {                              \
        constexpr int STK = 64;           \
        __VA_ARGS__;                      \
    }

struct Cands {
    int64_t n = 0;
    Scratch keys, k, seq, img;
    CandView view() const {
        CandView v;
        v.k = k.as<int32_t>();
        v.seq = seq.as<int32_t>();
        v.img = img.as<double>();
        v.n = n;
        return v;
    }
};

static int stack_depth_for(const Scene& s, bool brute)
{
    return (brute || std::max(s.max_depth, s.walk_depth) < 31) ? 32 : 64;
}

struct PathSet {
    int64_t n = 0;
    Scratch cells, valid, amp, len, recs, rstart;
};

// One source's candidate pipeline, split where the host needs a size.
struct Branch {
    const double* src = nullptr;
    const double* hemi = nullptr;
    int which = 0;
    hipStream_t st = nullptr;
    int64_t* d_cnt = nullptr;
    unsigned long long* d_app = nullptr;
    Scratch keys;
    int64_t nkeys = 0;
    Cands cd;
    PathSet ps;
    // hash set: 0 sized from the last call's count, 1 the standard set,
    // 2 sized for every prefix being distinct (after overflows)
    int table_level = 0;
    Scratch table;            // the hash set of the next phase A (cleared), cap slots
    int64_t cap = 0;
    uint64_t max_probe = 0;
    Scratch mask;             // geometric validity, R rows of n_words 32-bit words
    int64_t n_words = 0;
    unsigned long long* d_work = nullptr;   // counting build: node visits, triangle tests of discovery
    hipEvent_t ev_disc[2] = {nullptr, nullptr};   // around the discovery kernel (stage times only)
};

// RIS description for the kernels
static RisView make_ris_view(const TraceArgs& a)
{
    RisView rv;
    rv.M = (int32_t)a.ris->M;
    rv.pad = 0;
    rv.elem = a.ris->elem.as<double>();
    rv.order = a.ris->order.as<int32_t>();
    for (int q = 0; q < 3; ++q) {
        rv.centre[q] = a.ris->centre[q];
        rv.normal[q] = a.ris->normal[q];
    }
    rv.normal_norm = sqrt(rv.normal[0] * rv.normal[0] + rv.normal[1] * rv.normal[1] + rv.normal[2] * rv.normal[2]);
    rv.dy = a.ris->dy;
    rv.dz = a.ris->dz;
    rv.gain = a.ris->gain > 0 ? a.ris->gain
                              : 4.0 * 3.141592653589793 * a.ris->dy * a.ris->dz / (a.tc.lambda * a.tc.lambda);
    rv.q = a.ris->q;
    return rv;
}

// The field reaching every element (TxmRec per element, in txm): the direct
// leg, and with `incoming` the reflections Tx -> surfaces -> element for the
// Tx candidates valid at the RIS centre.  Launched on stream si (beside the
// path kernels); its scratch lives on si.
template <int KM>
static void ris_incident(Ctx& c, const SceneView& sv, int stk, const TraceArgs& a, bool brute, bool incoming,
                         const Branch& bt, const RisView& rv, unsigned long long* d_ctr, TxmRec* txm, hipStream_t si)
{
    const int64_t M = rv.M;
    unsigned long long* d_legs = d_ctr + 1;
    SEL_BOOL(brute, BR,
             SEL_STK(stk, hipLaunchKernelGGL((k_txm<BR, STK>), dim3(nblk(M, 64)), dim3(64), 0, si, sv, a.tc, rv, txm,
                                             d_legs)));
    HIP_CHECK(hipGetLastError());
    if (!incoming || M == 0 || bt.cd.n == 0) return;
    // sequences valid from the Tx to the RIS centre, then every (sequence, element)
    const int64_t nc = bt.cd.n;
    Scratch in_ok(c, (size_t)nc, si), in_off(c, sizeof(int64_t) * (size_t)nc, si),
        in_list(c, sizeof(int32_t) * (size_t)nc, si);
    int64_t* d_nin = (int64_t*)(d_ctr + 16);
    SEL_BOOL(brute, BR,
             SEL_STK(stk, hipLaunchKernelGGL((k_in_centre<BR, STK, KM>), dim3(nblk(nc, LEG_B)), dim3(LEG_B), 0, si, sv,
                                             bt.cd.view(), a.tc.tx[0], a.tc.tx[1], a.tc.tx[2], rv.centre[0],
                                             rv.centre[1], rv.centre[2], in_ok.as<uint8_t>(), d_legs)));
    HIP_CHECK(hipGetLastError());
    scan_flags(c, in_ok.as<uint8_t>(), in_off.as<int64_t>(), nc, d_nin, si);
    hipLaunchKernelGGL(k_in_list, dim3(nblk(nc, 256)), dim3(256), 0, si, in_ok.as<uint8_t>(), in_off.as<int64_t>(),
                       nc, in_list.as<int32_t>());
    HIP_CHECK(hipGetLastError());
    // launched for every candidate (no size read-back); rows past the list's length exit
    if (nc > ((int64_t)1 << 40) / M) throw inval_error("candidates x elements too large");
    Scratch contrib(c, sizeof(float2) * (size_t)(nc * M), si), emitted(c, (size_t)(nc * M), si);
    SEL_BOOL(brute, BR,
             SEL_STK(stk, hipLaunchKernelGGL((k_in_elem<BR, STK, KM>), dim3(nblk(nc * M, LEG_B)), dim3(LEG_B), 0, si, sv,
                                             bt.cd.view(), a.tc, rv, in_list.as<int32_t>(), d_nin,
                                             contrib.as<float2>(), emitted.as<uint8_t>(), d_legs, d_ctr + 17)));
    HIP_CHECK(hipGetLastError());
    hipLaunchKernelGGL(k_in_sum, dim3(nblk(M, 128)), dim3(128), 0, si, contrib.as<float2>(), emitted.as<uint8_t>(),
                       d_nin, M, txm);
    HIP_CHECK(hipGetLastError());
}

// 64-bit words per candidate key: one up to order 3, two for orders 4 and 5
static inline int key_words(int K) { return K > RT_KM_SMALL ? 2 : 1; }
// end of the key bits: 21 per surface, orders above 3 continue in word 1
static inline int key_end_bit(int K) { return K > RT_KM_SMALL ? 64 + RT_KEY_BITS * (K - 3) : RT_KEY_BITS * K; }

// Phase A of the candidates: discovery rays, prefix keys into a hash set,
// occupied slots compacted behind a leading 0 (the empty sequence); the
// count is left in d_app[0] (overflow flag in d_app[1]).  Exhaustive mode:
// every surface sequence, sorted and de-duplicated (count in d_cnt).
// The hash set of a branch's phase A, allocated on `st` (not cleared): probe
// runs of at most 256 (an overflow makes the caller repeat with the next
// level): first a set of at least 4x the last call's unique count, then 2^20
// slots, then at least 2 x (keys + 1) slots, at most 2^27, with unbounded
// probing.
static void prepare_table(Ctx& c, const TraceArgs& a, Branch& br, hipStream_t st)
{
    const int64_t rows = br.hemi ? 2 * a.n_rays : a.n_rays;
    const int64_t want = 2 * rows * a.tc.K + 2;
    auto set_size = [want](int64_t limit) {
        int64_t cap = 1024;
        while (cap < want && cap < limit) cap <<= 1;
        return cap;
    };
    int64_t cap = set_size(br.table_level == 2 ? ((int64_t)1 << 27) : ((int64_t)1 << 20));
    if (br.table_level == 0) {
        const int64_t h = c.cand_hint[br.which].load();
        int64_t l = 1024;
        while (h > 0 && l < 4 * h && l < cap) l <<= 1;
        if (h > 0 && l < cap)
            cap = set_size(l);
        else
            br.table_level = 1;   // no smaller set: an overflow goes straight to the last level
    }
    br.cap = cap;
    br.max_probe = br.table_level == 2 ? (uint64_t)(cap - 1) : (uint64_t)255;
    br.table = Scratch(c, sizeof(unsigned long long) * (size_t)key_words(a.tc.K) * (size_t)cap, st);
}

template <int KM>
static void cand_phase_a(Ctx& c, const SceneView& sv, int stk, const TraceArgs& a, bool brute, bool exhaustive,
                         bool keep_hits, Channel& ch, Branch& br, unsigned long long* d_segs)
{
    const int K = a.tc.K;
    constexpr int W = KM > RT_KM_SMALL ? 2 : 1;
    hipStream_t st = br.st;
    if (exhaustive) {
        int64_t ns = sv.n_surf;
        int64_t total = 0, p = 1;
        for (int k = 1; k <= K; ++k) {
            p *= ns;
            total += p;
            if (total > (int64_t)1 << 26) throw inval_error("exhaustive candidate set too large");
        }
        int64_t nkeys = total + 1;
        Scratch keys(c, sizeof(uint64_t) * W * (size_t)nkeys, st), sorted(c, sizeof(uint64_t) * W * (size_t)nkeys, st);
        HIP_CHECK(hipMemsetAsync(keys.p, 0, keys.bytes, st));
        if (total > 0)
            hipLaunchKernelGGL(k_exhaustive_keys<W>, dim3(nblk(total, 256)), dim3(256), 0, st, ns, K, total,
                               keys.as<uint64_t>());
        HIP_CHECK(hipGetLastError());
        sort_keys(c, keys.as<uint64_t>(), sorted.as<uint64_t>(), nkeys, W, 0, key_end_bit(K), st);
        br.keys = Scratch(c, sizeof(uint64_t) * W * (size_t)nkeys, st);
        unique_keys(c, sorted.as<uint64_t>(), br.keys.as<uint64_t>(), nkeys, W, br.d_cnt, st);
        return;
    }
    const double* src = br.src;
    const double* hemi_n = br.hemi;
    int64_t rows = hemi_n ? 2 * a.n_rays : a.n_rays;
    if (rows > ((int64_t)1 << 31)) throw inval_error("too many discovery rays");
    // hit lists are written only when the caller keeps them
    Scratch hits(c, keep_hits ? sizeof(int32_t) * (size_t)(rows * K) : 0, st);
    if (keep_hits && rows > 0 && K > 0) {
        hipLaunchKernelGGL(k_fill_neg, dim3(nblk(rows * K, 256)), dim3(256), 0, st, hits.as<int32_t>(), rows * K);
        HIP_CHECK(hipGetLastError());
    }
    if (!br.table.p) {
        prepare_table(c, a, br, st);
        clear3(br.table.as<uint64_t>(), (int64_t)(br.table.bytes / 8), nullptr, 0, nullptr, 0, st);
    }
    Scratch table = std::move(br.table);
    table.st = st;   // released on the branch's stream after its last reader
    const int64_t cap = br.cap;
    const uint64_t max_probe = br.max_probe;
    if (rows > 0 && K > 0 && sv.n_tri > 0) {
        const int32_t *perm, *off;
        fib_tables(c, &perm, &off);
        const int64_t n_launch = (rows + RT_FIB_CHUNK - 1) / RT_FIB_CHUNK * RT_FIB_CHUNK;
        const bool count = (a.tc.flags & 16) != 0 && !brute;
        if (br.ev_disc[0]) HIP_CHECK(hipEventRecord(br.ev_disc[0], st));
        if (!brute && !count && sparse_rays(a.n_rays, sv.n_tri, K)) {
            SEL_STK(stk, hipLaunchKernelGGL((k_discover_quad<STK, KM>), dim3(nblk(4 * n_launch, DISC_B)), dim3(DISC_B),
                                            0, st, sv, src[0], src[1], src[2], perm, off, rows, hemi_n ? 1 : 0,
                                            hemi_n ? hemi_n[0] : 0.0, hemi_n ? hemi_n[1] : 0.0,
                                            hemi_n ? hemi_n[2] : 0.0, K, keep_hits ? hits.as<int32_t>() : nullptr,
                                            d_segs, table.as<unsigned long long>(), (uint64_t)(cap - 1), max_probe,
                                            (int*)(br.d_app + 1)));
        } else {
            SEL_BOOL(brute, BR, SEL_BOOL(count, CN,
                     SEL_STK(stk, hipLaunchKernelGGL((k_discover<BR, STK, KM, CN>), dim3(nblk(n_launch, DISC_B)),
                                                     dim3(DISC_B), 0, st, sv, src[0], src[1], src[2], perm, off, rows,
                                                     hemi_n ? 1 : 0, hemi_n ? hemi_n[0] : 0.0, hemi_n ? hemi_n[1] : 0.0,
                                                     hemi_n ? hemi_n[2] : 0.0, K, keep_hits ? hits.as<int32_t>() : nullptr,
                                                     d_segs, table.as<unsigned long long>(), (uint64_t)(cap - 1), max_probe,
                                                     (int*)(br.d_app + 1), br.d_work))));
        }
        HIP_CHECK(hipGetLastError());
        if (br.ev_disc[1]) HIP_CHECK(hipEventRecord(br.ev_disc[1], st));
    }
    if (keep_hits) {
        ch.n_hits_rows[br.which] = rows;
        ch.hits[br.which] = std::move(hits);
    }
    br.keys = Scratch(c, sizeof(uint64_t) * W * (size_t)(cap + 1), st);
    if (W == 1)
        hipLaunchKernelGGL(k_table_compact, dim3(nblk(cap, TC_B * TC_PT)), dim3(TC_B), 0, st,
                           table.as<unsigned long long>(), cap, br.keys.as<uint64_t>(), cap, br.d_app);
    else
        hipLaunchKernelGGL(k_table_compact2, dim3(nblk(cap, TC_B * TC_PT)), dim3(TC_B), 0, st,
                           table.as<unsigned long long>(), cap, br.keys.as<uint64_t>(), cap, br.d_app);
    HIP_CHECK(hipGetLastError());
}

// Size read-back after phase A: number of unique candidates (incl. order 0),
// or -1 if the hash set overflowed below the last level.
static int64_t cand_count(Ctx& c, const Branch& br, bool exhaustive)
{
    if (exhaustive) return read_i64(br.d_cnt, br.st);
    int64_t hq[2];
    read_i64s((const int64_t*)br.d_app, hq, 2, br.st);
    if (hq[1] & 1) {
        if (br.table_level < 2) return -1;   // repeat phase A with the next set
        throw inval_error("candidate hash set overflow");
    }
    c.cand_hint[br.which].store(hq[0] + 1);
    return hq[0] + 1;
}

// Phase B: the unique keys in key order (the canonical candidate order).
// Returns their number: n for one-word keys (the hash set holds each once);
// two-word keys may have been inserted twice (see hash_insert2), so they are
// de-duplicated after the sort and counted again (one more size read-back).
static int64_t cand_phase_b(Ctx& c, const TraceArgs& a, bool exhaustive, Branch& br, int64_t n)
{
    if (exhaustive) return n;
    const int W = key_words(a.tc.K);
    Scratch sorted(c, sizeof(uint64_t) * W * (size_t)(n > 0 ? n : 1), br.st);
    sort_keys(c, br.keys.as<uint64_t>(), sorted.as<uint64_t>(), n, W, 0, key_end_bit(a.tc.K), br.st);
    if (W == 1) {
        br.keys = std::move(sorted);
        return n;
    }
    br.keys = Scratch(c, sizeof(uint64_t) * W * (size_t)(n > 0 ? n : 1), br.st);
    unique_keys(c, sorted.as<uint64_t>(), br.keys.as<uint64_t>(), n, W, br.d_cnt, br.st);
    const int64_t nu = read_i64(br.d_cnt, br.st);
    c.cand_hint[br.which].store(nu);
    return nu;
}

// candidate images and the geometric test of every (receiver, candidate) cell
template <int KM>
static void geo_launch(Ctx& c, const SceneView& sv, const TraceArgs& a, Branch& br, int64_t n_cand,
                       const uint64_t* rx_order)
{
    hipStream_t st = br.st;
    Cands& cd = br.cd;
    cd.n = n_cand;
    cd.keys = std::move(br.keys);
    cd.k = Scratch(c, sizeof(int32_t) * (size_t)n_cand, st);
    cd.seq = Scratch(c, sizeof(int32_t) * KM * (size_t)n_cand, st);
    cd.img = Scratch(c, sizeof(double) * 3 * KM * (size_t)n_cand, st);
    hipLaunchKernelGGL(k_cand_prep<KM>, dim3(nblk(n_cand, 128)), dim3(128), 0, st, cd.keys.as<uint64_t>(), n_cand, sv,
                       br.src[0], br.src[1], br.src[2], cd.k.as<int32_t>(), cd.seq.as<int32_t>(),
                       cd.img.as<double>());
    HIP_CHECK(hipGetLastError());
    const int64_t R = a.R;
    if (R > 0 && n_cand > ((int64_t)1 << 40) / R) throw inval_error("receivers x candidates too large for one call");
    if (nblk(R, 64) > 65535 || n_cand > 0x7fffffff) throw inval_error("receiver or candidate count too large");
    const int64_t n_words = (n_cand + 31) / 32;
    br.n_words = n_words;
    br.mask = Scratch(c, sizeof(uint32_t) * (size_t)(R * n_words), st);
    if (R * n_words > 0) {
        hipLaunchKernelGGL(k_geo_mask<KM>, dim3((unsigned)n_words, nblk(R, 64)), dim3(GEO_B), 0, st, sv, cd.view(),
                           br.src[0], br.src[1], br.src[2], a.rx_dev, rx_order, R, n_words,
                           br.mask.as<uint32_t>());
        HIP_CHECK(hipGetLastError());
    }
    // receivers' offsets into the valid cells; entry R = total
    Scratch cnt(c, sizeof(int64_t) * (size_t)(R + 1), st);
    br.ps.rstart = Scratch(c, sizeof(int64_t) * (size_t)(R + 1), st);
    hipLaunchKernelGGL(k_cell_count, dim3(nblk(R + 1, 4)), dim3(256), 0, st, br.mask.as<uint32_t>(), R, n_words,
                       cnt.as<int64_t>());
    HIP_CHECK(hipGetLastError());
    scan_i64(c, cnt.as<int64_t>(), br.ps.rstart.as<int64_t>(), R + 1, nullptr, st);
}

// the valid cells in (receiver, candidate) order, legs and field of each path
template <int KM>
static void paths_launch(Ctx& c, const SceneView& sv, int stk, const TraceArgs& a, bool brute, bool field,
                         Branch& br, int64_t n, unsigned long long* d_segs, unsigned long long* d_valid)
{
    hipStream_t st = br.st;
    PathSet& ps = br.ps;
    const int64_t R = a.R;
    ps.n = n;
    ps.cells = Scratch(c, sizeof(uint64_t) * (size_t)(n > 0 ? n : 1), st);
    if (n > 0) {
        hipLaunchKernelGGL(k_cell_emit, dim3(nblk(R, 4)), dim3(256), 0, st, br.mask.as<uint32_t>(), R, br.n_words,
                           br.cd.n, ps.rstart.as<int64_t>(), ps.cells.as<uint64_t>());
        HIP_CHECK(hipGetLastError());
    }
    br.mask.release();
    ps.valid = Scratch(c, (size_t)(n > 0 ? n : 1), st);
    ps.recs = Scratch(c, sizeof(PathRec<KM>) * (size_t)(n > 0 ? n : 1), st);
    if (field) {
        ps.amp = Scratch(c, sizeof(float2) * (size_t)(n > 0 ? n : 1), st);
        ps.len = Scratch(c, sizeof(double) * (size_t)(n > 0 ? n : 1), st);
    }
    if (n == 0) return;
    CandView cv = br.cd.view();
    const double* src = br.src;
    SEL_BOOL(brute, BR,
             SEL_BOOL(field, FI,
                      SEL_STK(stk, hipLaunchKernelGGL((k_paths<BR, FI, STK, KM>), dim3(nblk(n, LEG_B)), dim3(LEG_B), 0,
                                                      st, sv, cv, a.tc, src[0], src[1], src[2], a.rx_dev,
                                                      ps.cells.as<uint64_t>(), n, ps.valid.as<uint8_t>(),
                                                      ps.amp.as<float2>(), ps.len.as<double>(),
                                                      ps.recs.as<PathRec<KM>>(), d_segs, d_valid))));
    HIP_CHECK(hipGetLastError());
}

struct StageTimer {
    bool on;
    hipStream_t st;
    bool all;   // every stage, or only the marks that bracket the per-element kernel
    std::vector<hipEvent_t> ev;   // per mark, null where not recorded
    StageTimer(bool o, bool every, hipStream_t s) : on(o), st(s), all(every) {}
    // every event is a marker the device processes between kernels: record only what is asked for
    void mark(bool per_element = false, hipStream_t on_stream = nullptr) {
        hipEvent_t e = nullptr;
        if (on && (all || per_element)) {
            HIP_CHECK(hipEventCreate(&e));
            HIP_CHECK(hipEventRecord(e, on_stream ? on_stream : st));
        }
        ev.push_back(e);
    }
    ~StageTimer() {
        for (auto e : ev)
            if (e) (void)hipEventDestroy(e);
    }
};

struct Event {
    hipEvent_t e = nullptr;
    Event() { HIP_CHECK(hipEventCreateWithFlags(&e, hipEventDisableTiming)); }
    ~Event() { (void)hipEventDestroy(e); }
    Event(const Event&) = delete;
    Event& operator=(const Event&) = delete;
};

// A buffer that two streams read: an error on the way waits for both before
// the buffer, declared ahead of this, goes back.
struct DrainOnError {
    hipStream_t a, b;
    int n = std::uncaught_exceptions();
    DrainOnError(hipStream_t a_, hipStream_t b_) : a(a_), b(b_) {}
    ~DrainOnError()
    {
        if (std::uncaught_exceptions() > n) {
            (void)hipStreamSynchronize(a);
            (void)hipStreamSynchronize(b);
        }
    }
    DrainOnError(const DrainOnError&) = delete;
    DrainOnError& operator=(const DrainOnError&) = delete;
};

// events that can time the kernels between them
struct TimedEvent {
    hipEvent_t e = nullptr;
    TimedEvent() { HIP_CHECK(hipEventCreate(&e)); }
    ~TimedEvent() { (void)hipEventDestroy(e); }
    TimedEvent(const TimedEvent&) = delete;
    TimedEvent& operator=(const TimedEvent&) = delete;
};

template <int KM>
static void trace_km(Ctx& c, const TraceArgs& a, Channel& ch, TraceOut& out, bool timing, hipStream_t st)
{
    const SceneView sv = a.scene->view();
    const bool brute = (a.tc.flags & 4) != 0;
    const bool keep_hits = (a.tc.flags & 1) != 0;
    const bool keep_paths = (a.tc.flags & 2) != 0;
    const bool exhaustive = (a.tc.flags & 8) != 0;
    const bool count_work = (a.tc.flags & 16) != 0;
    const bool incoming = (a.tc.flags & 32) != 0;   // reflections Tx -> surfaces -> element
    const bool fresnel = a.tc.fresnel != 0;
    const bool keep_cir = (a.tc.flags & 256) != 0;   // per-path delays and amplitudes for rt_cir
    const int stk = stack_depth_for(*a.scene, brute);
    const int64_t R = a.R;
    const int64_t M = a.ris ? a.ris->M : 0;
    ch.R = R;
    ch.M = M;
    ch.K = a.tc.K;
    StageTimer tm(timing, (a.tc.flags & 512) != 0, st);
    tm.mark();   // 0

    // counters: [0] discovery segments, [1] leg segments, [2..4] Tx count / append / hash overflow,
    // [5..7] centre count / append / hash overflow, [8..12] work of the counting build,
    // [13] valid environment paths, [14] per-element slots whose grouped leg walk fell back,
    // [15] discovery segments of a repeated phase A (not reported)
    // 0 discovery segments, 1 legs, 2-4 Tx branch counts, 5-7 centre branch counts,
    // 8-12 work, 13 env paths, 14 leg-walk fallbacks, 15 dummy segments,
    // 16 incoming sequences, 17 incoming element paths
    // 18-20, 21-23: node visits, triangle tests, segments of the counting discovery build (Tx, centre)
    Scratch ctr(c, 8 * 24, st);
    unsigned long long* d_ctr = ctr.as<unsigned long long>();
    unsigned long long* d_disc = d_ctr;
    unsigned long long* d_legs = d_ctr + 1;
    unsigned long long* d_work = d_ctr + 8;
    // the counting builds walk the scene's Morton tree
    SceneView svc = sv;
    Scratch lbvh;
    if (count_work && !brute && sv.n_tri > 1) {
        lbvh_nodes(c, *a.scene, lbvh, st);
        svc.nodes = lbvh.as<float4>();
        svc.root = 0;
    }
    ch.E_env = Scratch(c, sizeof(float2) * (size_t)R, st);
    Scratch uptr, useq;
    if (a.ris) uptr = Scratch(c, sizeof(int64_t) * (size_t)(R + 1), st);
    tm.mark();   // 1

    // the Tx branch runs on `st`, the RIS-centre branch on a side stream
    Branch bt, bu;
    bt.src = a.tc.tx;
    bt.which = 0;
    bt.st = st;
    bt.d_cnt = (int64_t*)(d_ctr + 2);
    bt.d_app = d_ctr + 3;
    bt.d_work = d_ctr + 18;
    const bool time_disc = timing && (a.tc.flags & 512) != 0;
    std::unique_ptr<TimedEvent[]> ev_d(time_disc ? new TimedEvent[4] : nullptr);   // created only when asked for
    if (time_disc) {
        bt.ev_disc[0] = ev_d[0].e;
        bt.ev_disc[1] = ev_d[1].e;
    }
    const bool two = a.ris != nullptr;
    Event fork, join;
    SideStream side(c);   // returned to the pool after the join below
    if (two) {
        bu.src = a.ris->centre;
        bu.hemi = a.ris->normal;
        bu.which = 1;
        bu.st = side.s;
        bu.d_cnt = (int64_t*)(d_ctr + 5);
        bu.d_app = d_ctr + 6;
        bu.d_work = d_ctr + 21;
        if (time_disc) {
            bu.ev_disc[0] = ev_d[2].e;
            bu.ev_disc[1] = ev_d[3].e;
        }
    }
    // the counters and both hash sets are cleared here, ahead of either discovery (a clear queued
    // behind the other branch's discovery waits for free compute units)
    if (!exhaustive) {
        prepare_table(c, a, bt, st);
        if (two) prepare_table(c, a, bu, st);
    }
    clear3(ctr.as<uint64_t>(), 24, bt.table.as<uint64_t>(), (int64_t)(bt.table.bytes / 8), bu.table.as<uint64_t>(),
           (int64_t)(bu.table.bytes / 8), st);
    HIP_CHECK(hipEventRecord(fork.e, st));
    if (two) HIP_CHECK(hipStreamWaitEvent(bu.st, fork.e, 0));
    // The receivers in Morton order of their positions, for the geometry kernel: on the centre
    // branch's stream, ahead of the discoveries (25 us of a lone workgroup for 64 x 64 receivers,
    // that would wait for a free compute unit behind them; the Tx branch is the one that the
    // first geometry waits for).  A few receivers go as they come: at most 4 waves of them a
    // candidate, and two launches and a wait cost 20 us of the 350 of a small trace.  Among
    // 1900 to 100 000 triangles (rooms and office floors, orders 2 to 5, receivers drawn or on a
    // grid) no trace of 32 to 256 receivers was slower than with the sort.
    if (R >= ((int64_t)1 << RX_IDX_BITS)) throw inval_error("too many receivers");
    Scratch rx_order;
    DrainOnError drain(st, two ? bu.st : st);
    Event rx_ready;
    if (R > RX_SORT_MIN) {
        hipStream_t sx = two ? bu.st : st;
        rx_order = Scratch(c, sizeof(uint64_t) * (size_t)R, sx);
        Scratch rx_keys(c, sizeof(uint64_t) * (size_t)R, sx);
        const int bits = rx_axis_bits(R);
        hipLaunchKernelGGL(k_rx_keys, dim3(nblk(R, 256)), dim3(256), 0, sx, a.rx_dev, R, a.scene->box.as<float>(),
                           bits, rx_keys.as<uint64_t>());
        HIP_CHECK(hipGetLastError());
        sort_keys(c, rx_keys.as<uint64_t>(), rx_order.as<uint64_t>(), R, 1, RX_IDX_BITS, RX_IDX_BITS + 3 * bits, sx);
        if (two) HIP_CHECK(hipEventRecord(rx_ready.e, sx));
    }
    // 1-3: candidates
    cand_phase_a<KM>(c, svc, stk, a, brute, exhaustive, keep_hits, ch, bt, d_disc);
    if (two) cand_phase_a<KM>(c, svc, stk, a, brute, exhaustive, keep_hits, ch, bu, d_disc);
    // Each branch goes on as soon as its own count is back, so the Tx branch
    // (launched first) does not wait for the centre branch's discovery.  An
    // overflow of a hash set repeats phase A with the next level (the
    // discovery segments were counted by the first pass).
    unsigned long long* d_dummy = d_ctr + 15;
    auto count_of = [&](Branch& br) {
        int64_t n = cand_count(c, br, exhaustive);
        while (n < 0) {
            br.table_level += 1;
            HIP_CHECK(hipMemsetAsync(br.d_app, 0, 2 * sizeof(unsigned long long), br.st));
            cand_phase_a<KM>(c, svc, stk, a, brute, exhaustive, keep_hits, ch, br, d_dummy);
            n = cand_count(c, br, exhaustive);
        }
        return n;
    };
    const int64_t n_tx = cand_phase_b(c, a, exhaustive, bt, count_of(bt));
    tm.mark();   // 2
    // 4: geometry of every (receiver, candidate)
    if (two && R > RX_SORT_MIN) HIP_CHECK(hipStreamWaitEvent(st, rx_ready.e, 0));
    geo_launch<KM>(c, sv, a, bt, n_tx, rx_order.as<uint64_t>());
    const int64_t n_u0 = two ? cand_phase_b(c, a, exhaustive, bu, count_of(bu)) : 0;
    if (two) geo_launch<KM>(c, sv, a, bu, n_u0, rx_order.as<uint64_t>());
    out.n_cand_tx = n_tx;
    out.n_cand_u = n_u0;
    // the field reaching every element, on its own stream (forked here, launched
    // after the path kernels so that they go first)
    RisView rv{};
    Scratch txm;
    Event in_fork, in_ready;
    SideStream side_in(c);
    if (a.ris) {
        rv = make_ris_view(a);
        txm = Scratch(c, sizeof(TxmRec) * (size_t)rv.M, st);
        HIP_CHECK(hipEventRecord(in_fork.e, st));
        HIP_CHECK(hipStreamWaitEvent(side_in.s, in_fork.e, 0));
    }
    // 5-6: legs and fields
    const int64_t g_tx = read_i64(bt.ps.rstart.as<int64_t>() + R, st);
    paths_launch<KM>(c, sv, stk, a, brute, true, bt, g_tx, d_legs, d_ctr + 13);
    const int64_t g_u = two ? read_i64(bu.ps.rstart.as<int64_t>() + R, bu.st) : 0;
    if (two) paths_launch<KM>(c, sv, stk, a, brute, false, bu, g_u, d_legs, d_ctr + 13);
    if (a.ris) {
        ris_incident<KM>(c, sv, stk, a, brute, incoming, bt, rv, d_ctr, txm.as<TxmRec>(), side_in.s);
        HIP_CHECK(hipEventRecord(in_ready.e, side_in.s));
    }

    // environment field per receiver (Tx branch)
    {
        PathSet& ps = bt.ps;
        if (R > 0) {
            hipLaunchKernelGGL(k_env_reduce, dim3(nblk(R, ENV_B / 64)), dim3(ENV_B), 0, st, ps.rstart.as<int64_t>(), R,
                               ps.valid.as<uint8_t>(), ps.amp.as<float2>(), ch.E_env.as<float2>());
            HIP_CHECK(hipGetLastError());
        }
        if (keep_paths) {
            Scratch off2(c, sizeof(int64_t) * (size_t)(ps.n > 0 ? ps.n : 1), st);
            scan_flags(c, ps.valid.as<uint8_t>(), off2.as<int64_t>(), ps.n, (int64_t*)(d_ctr + 13), st);
            const int64_t n_env = read_i64((const int64_t*)(d_ctr + 13), st);
            ch.env = Scratch(c, sizeof(EnvRec) * (size_t)n_env, st);
            if (ps.n > 0) {
                hipLaunchKernelGGL(k_env_compact<KM>, dim3(nblk(ps.n, 128)), dim3(128), 0, st, ps.recs.as<PathRec<KM>>(),
                                   bt.cd.view(), ps.valid.as<uint8_t>(), off2.as<int64_t>(), ps.amp.as<float2>(),
                                   ps.len.as<double>(), ps.n, ch.env.as<EnvRec>());
                HIP_CHECK(hipGetLastError());
            }
        }
        if (keep_cir) {   // the environment paths of every receiver, in record order
            ch.env_cells = ps.n;
            ch.env_rstart = std::move(ps.rstart);
            ch.env_valid = std::move(ps.valid);
            ch.env_amp = std::move(ps.amp);
            ch.env_len = std::move(ps.len);
        }
    }
    // sequences valid from the RIS centre, grouped by receiver (centre branch), and the
    // receivers' launch order (cost bits alone: the keys come in receiver order, the sort is stable)
    int64_t n_u = 0;
    Scratch order;
    if (two) {
        PathSet& ps = bu.ps;
        hipStream_t su = bu.st;
        if (R >= ((int64_t)1 << 32)) throw inval_error("too many receivers");
        Scratch cnt(c, sizeof(int64_t) * (size_t)(R + 1), su), cost(c, sizeof(uint64_t) * (size_t)(R > 0 ? R : 1), su);
        order = Scratch(c, sizeof(uint64_t) * (size_t)(R > 0 ? R : 1), su);
        hipLaunchKernelGGL(k_u_count<KM>, dim3(nblk(R + 1, 4)), dim3(256), 0, su, ps.rstart.as<int64_t>(),
                           ps.recs.as<PathRec<KM>>(), ps.valid.as<uint8_t>(), R, cnt.as<int64_t>(),
                           cost.as<uint64_t>());
        HIP_CHECK(hipGetLastError());
        scan_i64(c, cnt.as<int64_t>(), uptr.as<int64_t>(), R + 1, bu.d_cnt, su);
        // rows for every geometric path (an upper bound of the valid ones)
        useq = Scratch(c, sizeof(int32_t) * useq_stride(KM) * (size_t)(ps.n > 0 ? ps.n : 1), su);
        if (R > 0) {
            hipLaunchKernelGGL(k_u_emit<KM>, dim3(nblk(R, 4)), dim3(256), 0, su, ps.rstart.as<int64_t>(),
                               ps.recs.as<PathRec<KM>>(), bu.cd.view(), ps.valid.as<uint8_t>(), R, uptr.as<int64_t>(),
                               useq.as<int32_t>());
            HIP_CHECK(hipGetLastError());
            sort_keys(c, cost.as<uint64_t>(), order.as<uint64_t>(), R, 1, 32, 52, su);
        }
        if (keep_paths || keep_cir) n_u = read_i64(bu.d_cnt, su);
    }
    tm.mark();   // 3: the Tx branch's legs and field are queued on the caller's stream
    tm.mark();   // 4

    // The per-element kernel needs only the centre branch (its sequences per
    // receiver) and the field reaching the elements: it runs on the centre
    // branch's stream, beside the Tx branch's legs and field on the caller's
    // stream; the caller's stream joins it below.
    const hipStream_t sr = two ? bu.st : st;
    if (!a.ris) {
        ch.H = Scratch(c, 0, st);
        tm.mark();
        tm.mark();
    } else {
        HIP_CHECK(hipStreamWaitEvent(sr, in_ready.e, 0));   // the field reaching every element
        ch.H = Scratch(c, sizeof(float2) * (size_t)(R * M), sr);
        if (keep_paths) ch.ris_valid = Scratch(c, (size_t)((n_u + R) * M), sr);
        if (keep_paths || keep_cir) {
            ch.cir_amp = Scratch(c, sizeof(float2) * (size_t)((n_u + R) * M), sr);
            ch.cir_len = Scratch(c, sizeof(double) * (size_t)((n_u + R) * M), sr);
        }
        int n_mchunk = (int)((M + 63) / 64);
        int64_t waves = R * n_mchunk;
        int64_t threads = waves * 64;
        tm.mark(true, sr);   // 5
        if (threads > 0) {
            if (count_work && !brute && !keep_paths && !keep_cir) {
                SEL_STK(stk, hipLaunchKernelGGL((k_ris<false, false, STK, true, false, KM>), dim3(nblk(threads, RIS_B)),
                                                dim3(RIS_B), 0, sr, svc, a.tc, rv, txm.as<TxmRec>(), a.rx_dev, R,
                                                uptr.as<int64_t>(), useq.as<int32_t>(), order.as<uint64_t>(), n_mchunk, ch.H.as<float2>(),
                                                ch.ris_valid.as<uint8_t>(), (float2*)nullptr, (double*)nullptr, d_legs,
                                                d_work, d_ctr + 14));
            } else {
                SEL_BOOL(fresnel, FR, SEL_BOOL(brute, BR,
                         SEL_BOOL(keep_paths || keep_cir, KP,
                                  SEL_STK(stk, hipLaunchKernelGGL((k_ris<BR, KP, STK, false, FR, KM>),
                                                                  dim3(nblk(threads, RIS_B)), dim3(RIS_B), 0, sr, sv,
                                                                  a.tc, rv, txm.as<TxmRec>(), a.rx_dev, R,
                                                                  uptr.as<int64_t>(), useq.as<int32_t>(),
                                                                  order.as<uint64_t>(), n_mchunk, ch.H.as<float2>(),
                                                                  keep_paths ? ch.ris_valid.as<uint8_t>() : nullptr,
                                                                  ch.cir_amp.as<float2>(), ch.cir_len.as<double>(),
                                                                  d_legs, d_work, d_ctr + 14)))));
            }
        }
        HIP_CHECK(hipGetLastError());
        tm.mark(true, sr);   // 6
        if (keep_paths) {
            ch.n_u = n_u;
            ch.useq = std::move(useq);
        }
        if (keep_cir) ch.cir_uptr = std::move(uptr);
    }
    if (two) {   // the caller's stream joins the centre branch (and the per-element kernel)
        HIP_CHECK(hipEventRecord(join.e, sr));
        HIP_CHECK(hipStreamWaitEvent(st, join.e, 0));
    }
    ch.key_words = key_words(a.tc.K);
    ch.useq_stride = useq_stride(KM);
    if (keep_paths || keep_hits) {   // the candidate keys are small: kept with either flag
        ch.n_cand[0] = bt.cd.n;
        ch.cand_keys[0] = std::move(bt.cd.keys);
        if (two) {
            ch.n_cand[1] = bu.cd.n;
            ch.cand_keys[1] = std::move(bu.cd.keys);
        }
    }
    // temporaries of the centre branch are released on the main stream (after the join)
    if (two) {
        for (Scratch* p : {&bu.keys, &bu.cd.keys, &bu.cd.k, &bu.cd.seq, &bu.cd.img, &bu.ps.cells, &bu.ps.valid,
                           &bu.ps.amp, &bu.ps.len, &bu.ps.recs, &bu.ps.rstart})
            p->st = st;
        if (!keep_paths) useq.st = st;
        order.st = st;
        rx_order.st = st;
    }
    int64_t h[24];
    read_i64s((const int64_t*)d_ctr, h, 24, st);
    tm.mark();   // 7
    out.disc_segments = h[0];
    out.leg_segments = h[1];
    out.segments = h[0] + h[1];
    out.n_env = h[13];
    out.n_u = h[5];
    out.n_slots = a.ris ? h[5] + R : 0;
    ch.n_env = out.n_env;
    ch.n_slots = out.n_slots;
    ch.keep_cir = keep_cir;
    for (int q = 0; q < 5; ++q) out.work[q] = h[8 + q];
    out.leg_walk_fallbacks = h[14];
    out.n_in_seq = incoming && a.ris ? h[16] : 0;
    out.n_in_paths = incoming && a.ris ? h[17] : 0;
    for (int q = 0; q < 6; ++q) out.disc_work[q] = h[18 + q];
    if (time_disc) {   // the repeats of phase A after a hash-set overflow are not timed separately
        HIP_CHECK(hipStreamSynchronize(st));
        auto el = [&](int i, int j) {
            float ms = 0.0f;
            if (hipEventElapsedTime(&ms, ev_d[i].e, ev_d[j].e) != hipSuccess) {
                (void)hipGetLastError();
                return -1.0f;
            }
            return ms;
        };
        out.ms_disc[0] = fmaxf(el(0, 1), 0.0f);
        if (two) {
            out.ms_disc[1] = fmaxf(el(2, 3), 0.0f);
            // span of both launches: from the earlier start to the later end (the two streams overlap)
            const float start_gap = el(0, 2);   // > 0: the Tx launch started first
            const float t_first = start_gap >= 0.0f ? 0.0f : -start_gap;
            const float end_tx = t_first + out.ms_disc[0];
            const float end_u = (start_gap >= 0.0f ? start_gap : 0.0f) + out.ms_disc[1];
            out.ms_disc[2] = fmaxf(end_tx, end_u);
        } else {
            out.ms_disc[2] = out.ms_disc[0];
        }
    }
    if (timing) {
        HIP_CHECK(hipStreamSynchronize(st));
        auto el = [&](int i, int j) {
            float ms = 0;
            if (tm.ev[i] && tm.ev[j]) HIP_CHECK(hipEventElapsedTime(&ms, tm.ev[i], tm.ev[j]));
            return ms;
        };
        out.ms[0] = el(0, 1);                  // setup
        out.ms[1] = el(1, 2);                  // discovery + dedupe (both sources)
        out.ms[2] = 0.0f;
        out.ms[3] = el(2, 3);                  // Tx branch: images, paths, legs, field
        out.ms[4] = 0.0f;
        out.ms[5] = a.ris ? el(5, 6) : 0.0f;   // per-element kernel (k_ris) alone, on its stream
        out.ms[6] = a.ris ? el(2, 5) : 0.0f;   // from the candidates to the start of the per-element kernel
        out.ms[7] = el(0, 7);                  // total
    }
    ch.last_stream = st;
}

void trace(Ctx& c, const TraceArgs& a, Channel& ch, TraceOut& out, bool timing, hipStream_t st)
{
    if (a.tc.K <= RT_KM_SMALL)
        trace_km<RT_KM_SMALL>(c, a, ch, out, timing, st);
    else
        trace_km<RT_MAX_K>(c, a, ch, out, timing, st);
}

// --------------------------------------------------------------------------
// Channel impulse response of one configuration (delay bins of width
// L_bin / c), bin = floor(length / L_bin): the gamma-weighted amplitudes of a
// receiver's paths summed per bin.
// --------------------------------------------------------------------------
constexpr int CIR_B = 256;
constexpr int CIR_G = 3072;   // most bins of a pass (two 64-bit LDS counters each)

// Sum over the wave, in lane 63.
typedef int i32x2 __attribute__((ext_vector_type(2)));
template <int CTRL, int ROWS>
__device__ __forceinline__ long long dpp_add_i64(long long v)
{
    i32x2 x = __builtin_bit_cast(i32x2, v);
    if constexpr (ROWS == 0xF) {
        x[0] = __builtin_amdgcn_mov_dpp(x[0], CTRL, 0xF, 0xF, true);
        x[1] = __builtin_amdgcn_mov_dpp(x[1], CTRL, 0xF, 0xF, true);
    } else {
        x[0] = __builtin_amdgcn_update_dpp(0, x[0], CTRL, ROWS, 0xF, false);
        x[1] = __builtin_amdgcn_update_dpp(0, x[1], CTRL, ROWS, 0xF, false);
    }
    return v + __builtin_bit_cast(long long, x);
}
__device__ __forceinline__ long long wave_sum_i64(long long v)
{
    v = dpp_add_i64<0xB1, 0xF>(v);    // quads: neighbour, pair
    v = dpp_add_i64<0x4E, 0xF>(v);
    v = dpp_add_i64<0x124, 0xF>(v);   // rows of 16: rotate by 4, by 8
    v = dpp_add_i64<0x128, 0xF>(v);
    v = dpp_add_i64<0x142, 0xA>(v);   // row 0 to 1, 2 to 3
    return dpp_add_i64<0x143, 0xC>(v);   // rows 0-1 to 2-3
}

// gamma-weighted amplitude of a RIS record (FP64 of the FP32 inputs)
__device__ __forceinline__ void cir_weight(float2 a, float2 g, double& ar, double& ai)
{
    ar = (double)a.x * (double)g.x - (double)a.y * (double)g.y;
    ai = (double)a.x * (double)g.y + (double)a.y * (double)g.x;
}

// an integer of magnitude below 2^62
__device__ __forceinline__ long long cir_i64(double x)
{
    const double h = floor(x * 0x1p-32);
    const i32x2 v = {(int)(unsigned)__builtin_fma(h, -0x1p32, x), (int)h};
    return __builtin_bit_cast(long long, v);
}

// Two records a lane (`on` false: no path).
struct CirPair {
    float2 a[2], g[2];
    double len[2];
};
template <bool LEN>
__device__ __forceinline__ void cir_load(CirPair& p, int i, const float2* camp, const double* clen, const float2* gamma,
                                         int64_t cell, int m, bool on)
{
    p.a[i] = camp[cell];
    p.g[i] = gamma[m];
    if (LEN) p.len[i] = clen[cell];
    if (!on) p.a[i] = make_float2(0.0f, 0.0f);
}

// One workgroup per receiver.  The bins are summed in fixed point: every term
// is rounded to a multiple of 2^-S, where 2^S scales the receiver's sum of
// |re| + |im| below 2^61, and added as a 64-bit integer, so the result does not
// depend on the order of the additions (deterministic) and each term's rounding
// error is at most 2^-61 of that sum.
//
// A receiver's RIS records lie one behind the other, slot by slot and element
// by element, and its four waves take them 128 at a time: in one run (SLOT
// false), or a slot a step (88 to 128 elements, or two slots of 49 to 64, where
// that leaves few lanes empty and keeps the bins of a step few).  Elements of a slot lie within a few
// centimetres, so in wide bins most of the 128 fall into two or three: the wave
// sums up to ROUNDS bins one by one and one lane adds to each (64 lanes adding
// to one LDS word take turns); narrow bins and slots of few elements have the
// lanes add (ROUNDS 0).  `inv` is 1 / l_bin where a length over l_bin rounds
// correctly by it, 0 for the general division.  Bound by the vector
// instructions and the kept records (16 bytes each, the amplitudes read
// twice), the next 128 on their way while 128 are summed.  Measured in turn
// with a wave a slot throughout, and with a record and two additions a lane in
// one run without loads ahead, us a call:
//   35 slots of 127 elements at 4096 receivers, 400 bins of 0.25 ns  113 | 117 | 225
//   1600 receivers, 400 bins of 0.25 ns: 24 elements                  30 |  39 |  31
//     61 elements                                                     38 |  43 |  52
//     271 elements                                                   107 | 137 | 165
//   1000 bins of 0.1 ns: 24 elements                                  30 |  44 |  34
//     1027 elements                                                  369 | 520 | 673
//   one slot a receiver: 64 receivers x 3997 elements, 0.25 ns        32 |  78 |  32
//     4096 x 1027 elements, 3000 bins of 0.1 ns                       77 | 167 | 100
template <bool SLOT, int ROUNDS>
__global__ __launch_bounds__(CIR_B) void k_cir(const int64_t* env_rstart, const uint8_t* env_valid,
                                               const float2* env_amp, const double* env_len, const int64_t* uptr,
                                               const float2* camp, const double* clen, int64_t M_, const float2* gamma,
                                               double l_bin, double inv, int64_t n_bins, int gper, float2* cir)
{
    extern __shared__ unsigned long long acc[];   // 2 gper
    __shared__ double red[CIR_B / 64];
    const int64_t r = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t e0 = env_rstart ? env_rstart[r] : 0, e1 = env_rstart ? env_rstart[r + 1] : 0;
    const int64_t s0 = uptr ? uptr[r] + r : 0, s1 = uptr ? uptr[r + 1] + r + 1 : 0;
    // the scale: sum of |re| + |im| over the receiver's paths (inside the window or not), reduced in a
    // fixed order
    double sa = 0.0;
    for (int64_t j = e0 + tid; j < e1; j += CIR_B)
        if (env_valid[j]) sa += fabs((double)env_amp[j].x) + fabs((double)env_amp[j].y);
    // a wave's records, 128 at a time, the next ones on their way meanwhile
    constexpr int W = CIR_B / 64;
    auto walk = [&](auto with_len, auto use) {
        const int M = (int)M_;
        if (M <= 0 || s0 >= s1) return;
        // the lane's records: c and c + 64 of the receiver's n, m the element of the first (SLOT: elements m and
        // m + 64 of slot sl, or element m of slots sl and sl + W)
        const int64_t first = s0 * M, n = (s1 - s0) * M;
        int64_t c = wave * 128 + lane, sl = s0 + wave;
        int m = SLOT ? lane : (wave * 128 + lane) % M;
        const int half = SLOT ? 0 : 64 % M, step = SLOT ? 0 : W * 128 % M;
        const bool two = M <= 64;
        auto more = [&]() { return SLOT ? sl < s1 : c - lane < n; };
        auto load = [&](CirPair& p) {
            if (SLOT) {
                const bool in = two ? sl + W < s1 && m < M : m + 64 < M;
                const int m0 = m < M ? m : M - 1, m1 = two ? m0 : in ? m + 64 : M - 1;
                cir_load<with_len>(p, 0, camp, clen, gamma, sl * M + m0, m0, m < M);
                cir_load<with_len>(p, 1, camp, clen, gamma, (two && in ? sl + W : sl) * M + m1, m1, in);
                sl += two ? 2 * W : W;
            } else {
                const int m1 = m + half - (m + half >= M ? M : 0);
                cir_load<with_len>(p, 0, camp, clen, gamma, first + (c < n ? c : n - 1), m, c < n);
                cir_load<with_len>(p, 1, camp, clen, gamma, first + (c + 64 < n ? c + 64 : n - 1), m1, c + 64 < n);
                c += W * 128;
                m += step;
                m -= m >= M ? M : 0;
            }
        };
        if (!more()) return;
        CirPair p, q;
        load(p);
        for (;;) {
            const bool go = more();
            if (go) load(q);
            use(p);
            if (!go) break;
            p = q;
        }
    };
    walk(std::false_type{}, [&](const CirPair& p) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (p.a[i].x != 0.0f || p.a[i].y != 0.0f) {
                double ar, ai;
                cir_weight(p.a[i], p.g[i], ar, ai);
                sa += fabs(ar) + fabs(ai);
            }
    });
    for (int o = 32; o > 0; o >>= 1) sa += __shfl_xor(sa, o, 64);
    if (lane == 0) red[wave] = sa;
    __syncthreads();
    double total = 0.0;
    for (int w = 0; w < CIR_B / 64; ++w) total += red[w];
    // total * 2^S < 2^61 (S kept in the range where 2^S is a finite double)
    const int S = total > 0.0 ? min(1000, max(-1000, 60 - ilogb(total))) : 0;
    const double scale = ldexp(1.0, S), unscale = ldexp(1.0, -S);
    for (int64_t g0 = 0; g0 < n_bins; g0 += gper) {
        const int gn = (int)(n_bins - g0 < gper ? n_bins - g0 : gper);
        for (int i = tid; i < 2 * gn; i += CIR_B) acc[i] = 0ull;
        __syncthreads();
        // delay bin of a path in this pass, -1: outside
        auto bin_of = [&](double len) {
            const double bin = floor(inv != 0.0 ? div_by(len, l_bin, inv) : len / l_bin) - (double)g0;
            return bin >= 0.0 && bin < (double)gn ? (int)bin : -1;
        };
        auto add = [&](int bin, long long re, long long im) {
            atomicAdd(&acc[2 * bin], (unsigned long long)re);
            atomicAdd(&acc[2 * bin + 1], (unsigned long long)im);
        };
        for (int64_t j = e0 + tid; j < e1; j += CIR_B) {
            if (!env_valid[j]) continue;
            const int bin = bin_of(env_len[j]);
            if (bin >= 0)
                add(bin, (long long)rint((double)env_amp[j].x * scale), (long long)rint((double)env_amp[j].y * scale));
        }
        walk(std::true_type{}, [&](const CirPair& p) {
            int bin[2];
            long long re[2], im[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                bin[i] = p.a[i].x != 0.0f || p.a[i].y != 0.0f ? bin_of(p.len[i]) : -1;
                double ar, ai;
                cir_weight(p.a[i], p.g[i], ar, ai);
                re[i] = cir_i64(rint(ar * scale));
                im[i] = cir_i64(rint(ai * scale));
            }
            // the bins of the wave one by one, then lane by lane if there are many
            for (int k = 0; k < ROUNDS; ++k) {
                const int any = bin[0] >= 0 ? bin[0] : bin[1];
                const unsigned long long act = __ballot(any >= 0);
                if (!act) return;
                const int b0 = __builtin_amdgcn_readlane(any, __builtin_ctzll(act));
                const bool m0 = bin[0] == b0, m1 = bin[1] == b0;
                const long long tr = wave_sum_i64((m0 ? re[0] : 0) + (m1 ? re[1] : 0));
                const long long ti = wave_sum_i64((m0 ? im[0] : 0) + (m1 ? im[1] : 0));
                if (lane == 63) add(b0, tr, ti);
                if (m0) bin[0] = -1;
                if (m1) bin[1] = -1;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (bin[i] >= 0) add(bin[i], re[i], im[i]);
        });
        __syncthreads();
        for (int i = tid; i < gn; i += CIR_B)
            cir[r * n_bins + g0 + i] = make_float2((float)((double)(long long)acc[2 * i] * unscale),
                                                   (float)((double)(long long)acc[2 * i + 1] * unscale));
        __syncthreads();
    }
}

void cir(Ctx& c, const Channel& ch, const float* gamma, double bin_s, int64_t n_bins, float* out, hipStream_t st)
{
    (void)c;
    if (ch.R == 0 || n_bins == 0) return;
    const double l_bin = 299792458.0 * bin_s;
    const bool ris = ch.M > 0 && ch.cir_uptr.bytes > 0;
    // a length times the reciprocal, corrected, is the rounded quotient except for a divisor with all
    // fraction bits set, and away from the ends of the range
    uint64_t u;
    std::memcpy(&u, &l_bin, sizeof u);
    const bool by_inv = l_bin > 1e-100 && l_bin < 1e100 && (~u & 0xFFFFFFFFFFFFFull) != 0;
    // The bins in passes of equal size, LDS for one pass: of 3072 where a receiver has many records to walk again or
    // the receivers are too few to fill the chip, of 2048 (a third more workgroups a compute unit) elsewhere (4096
    // receivers of one slot, 3000 bins: 50 for 59 us; 1600 of 36 x 512 records: 290 for 233).
    const int64_t records = ris ? ch.n_slots * ch.M / ch.R : 0;
    const int64_t most = ch.R >= 1024 && records < 4000 ? 2048 : CIR_G;
    const int64_t passes = (n_bins + most - 1) / most;
    const int gper = (int)((n_bins + passes - 1) / passes);
    auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)ch.R), dim3(CIR_B), sizeof(unsigned long long) * 2 * (size_t)gper, st,
                           ch.env_cells > 0 ? ch.env_rstart.as<int64_t>() : nullptr, ch.env_valid.as<uint8_t>(),
                           ch.env_amp.as<float2>(), ch.env_len.as<double>(), ris ? ch.cir_uptr.as<int64_t>() : nullptr,
                           ch.cir_amp.as<float2>(), ch.cir_len.as<double>(), ris ? ch.M : 0, (const float2*)gamma, l_bin,
                           by_inv ? 1.0 / l_bin : 0.0, n_bins, gper, (float2*)out);
    };
    if (l_bin < 0.05 || ch.M <= 48)
        run(k_cir<false, 0>);
    else if (ch.M <= 64 || (ch.M >= 88 && ch.M <= 128))
        run(k_cir<true, 4>);
    else
        run(k_cir<false, 4>);
    HIP_CHECK(hipGetLastError());
}

}  // namespace rt
