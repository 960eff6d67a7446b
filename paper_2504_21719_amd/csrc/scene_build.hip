// scene_build.hip -- on-device LBVH construction for gfx950.
//
// Pipeline (all device work on the caller's stream, one read-back at the end):
//   bounds      validate indices / materials / finiteness, bounds of the
//               triangle AABB centres (per-thread, wavefront, block, then one
//               ordered-int atomic per block and bound)
//   morton      63-bit Morton code (21 bits per axis) of every AABB centre,
//               quantised with one scale for all axes (the largest extent)
//   radix sort  stable LSD sort of (code, triangle) pairs, 8 passes of 8 bits;
//               equal codes keep input order, and the Karras split below breaks
//               ties by index, so every key is effectively unique
//   gather      triangles, unit normals (computed in FP64), materials and AABBs
//               in Morton order, so that traversal touches nearby memory
//   box levels  AABBs of 16, 256, 4096, ... consecutive triangles
//   hierarchy   one thread per internal node finds its key range and split
//               from longest-common-prefix lengths (Karras, HPG 2012) and the
//               boxes of its two children, which are runs of consecutive
//               triangles, from the box levels
//   splits      few triangles: a second binary tree, split by surface area
//   4-wide      the wide nodes are found level by level from the root (lists) of
//               that or of the hierarchy, numbered by a scan and written
// An invalid mesh runs through all of it with a stand-in point for what cannot
// be read, so that the flags need no read-back of their own.
//
// The scene is one allocation; what the build needs besides lies in the part
// that the wide nodes fill last.  On 1.02 M triangles a build with its release
// took 4.9 ms: 3.3 ms in 21 allocations and frees, and the kernels 1.5 ms, half
// of it in a walk to the root per node, launches per tree level over all nodes
// and same-address atomics.  It takes 1.1 ms so, 0.75 ms of it in the kernels
// (latency-bound: the moved bytes would take about 0.1 ms).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstddef>
#include <cstring>
#include <string>

#include "rt_internal.h"

#define HIPCHK(x)                                            \
    do {                                                     \
        hipError_t _e = (x);                                 \
        if (_e != hipSuccess) {                              \
            cleanup();                                       \
            return rt_hip_fail(_e, #x);                      \
        }                                                    \
    } while (0)

namespace {

constexpr int kBlock = 256;
constexpr int kRsItems = 8;
constexpr int kRsTile = kBlock * kRsItems;

__device__ __forceinline__ unsigned f2ord(float f) {
    unsigned u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float ord2f(unsigned u) {
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}
float ord2f_host(unsigned u) {
    unsigned v = (u & 0x80000000u) ? (u & 0x7fffffffu) : ~u;
    float f;
    std::memcpy(&f, &v, 4);
    return f;
}

// Levels of wide nodes that the device state has room for: Karras nodes over
// 63-bit keys with ties broken by 32 index bits lie at most 95 deep, and a wide
// level spans at least one binary level.
constexpr int kMaxLevels = 128;
struct BuildState {
    unsigned lo[3], hi[3];             // ordered-int bounds of the AABB centres
    unsigned err;                      // 1 vertex index, 2 material id, 4 non-finite coordinate
    int max_depth;                     // deepest leaf
    unsigned n_wide;
    int n_small;                       // subtrees that k_sah_top left
    int next_level;                    // first level that k_wide_top left
    int count[kMaxLevels + 1];         // wide nodes per level
    unsigned totals[8][256];           // digit counts of the sort's passes
};

__global__ void k_build_init(BuildState* __restrict__ st, unsigned* __restrict__ flags, int64_t n_int) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t j = i; j < (int64_t)(sizeof(BuildState) / 4); j += step) ((unsigned*)st)[j] = j < 3 ? 0xffffffffu : 0u;
    for (int64_t j = i; j < n_int; j += step) flags[j] = 0u;
}

// The vertices of triangle t; the origin for indices out of range or
// non-finite coordinates.  Returns the error bits.
__device__ __forceinline__ unsigned load_tri(const float* __restrict__ V, int64_t n_v, const int32_t* __restrict__ F,
                                             int64_t t, float p[9]) {
    unsigned err = 0;
    bool fin = true;
    for (int a = 0; a < 3; a++) {
        const int32_t i = F[3 * t + a];
        const bool ok = i >= 0 && i < n_v;
        if (!ok) err |= 1u;
        for (int c = 0; c < 3; c++) {
            p[3 * a + c] = ok ? V[3 * (int64_t)i + c] : 0.0f;
            fin = fin && isfinite(p[3 * a + c]);
        }
    }
    if (!fin) {
        err |= 4u;
        for (int c = 0; c < 9; c++) p[c] = 0.0f;
    }
    return err;
}

__device__ __forceinline__ float tri_lo(const float p[9], int a) { return fminf(fminf(p[a], p[3 + a]), p[6 + a]); }
__device__ __forceinline__ float tri_hi(const float p[9], int a) { return fmaxf(fmaxf(p[a], p[3 + a]), p[6 + a]); }
__device__ __forceinline__ float tri_centre(const float p[9], int a) { return 0.5f * (tri_lo(p, a) + tri_hi(p, a)); }

__global__ void __launch_bounds__(kBlock) k_bounds(const float* __restrict__ V, int64_t n_v, const int32_t* __restrict__ F,
                                                   const int32_t* __restrict__ M, int32_t n_mat, int64_t n_tri,
                                                   BuildState* __restrict__ st) {
    __shared__ unsigned red[kBlock / 64][7];
    unsigned v[7] = {0xffffffffu, 0xffffffffu, 0xffffffffu, 0u, 0u, 0u, 0u};
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < n_tri; t += (int64_t)gridDim.x * kBlock) {
        float p[9];
        unsigned e = load_tri(V, n_v, F, t, p);
        const int32_t m = M[t];
        if (m < 0 || m >= n_mat) e |= 2u;
        v[6] |= e;
        if (e) continue;
        for (int a = 0; a < 3; a++) {
            const unsigned c = f2ord(tri_centre(p, a));
            v[a] = min(v[a], c);
            v[3 + a] = max(v[3 + a], c);
        }
    }
    for (int off = 32; off >= 1; off >>= 1)
        for (int k = 0; k < 7; k++) {
            const unsigned o = __shfl_xor(v[k], off);
            v[k] = k < 3 ? min(v[k], o) : k < 6 ? max(v[k], o) : (v[k] | o);
        }
    if ((threadIdx.x & 63) == 0)
        for (int k = 0; k < 7; k++) red[threadIdx.x >> 6][k] = v[k];
    __syncthreads();
    if (threadIdx.x < 7) {
        const int k = threadIdx.x;
        unsigned r = red[0][k];
        for (int w = 1; w < kBlock / 64; w++) r = k < 3 ? min(r, red[w][k]) : k < 6 ? max(r, red[w][k]) : (r | red[w][k]);
        if (k < 3) atomicMin(&st->lo[k], r);
        else if (k < 6) atomicMax(&st->hi[k - 3], r);
        else if (r) atomicOr(&st->err, r);
    }
}

__device__ __forceinline__ uint64_t spread21(uint32_t v) {
    uint64_t x = v & 0x1fffffu;
    x = (x | (x << 32)) & 0x001f00000000ffffull;
    x = (x | (x << 16)) & 0x001f0000ff0000ffull;
    x = (x | (x << 8)) & 0x100f00f00f00f00full;
    x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

// One scale for all three axes, from the largest extent of the centres' box:
// the codes then split the longest axis first and keep splitting it until the
// cells are about as long as the shorter axes are, so a flat scene (2 x 2 km of
// terrain, tens of metres high) is not cut by height near the root.  On the
// 1.02 M-triangle scene this takes a third of the node visits off the
// traversal against a scale per axis.
// Also counts the digits of all keys for every pass of the sort (in the passes'
// own histograms the same sums cost 5 us a pass in same-address atomics).
__global__ void __launch_bounds__(kBlock) k_morton(const float* __restrict__ V, int64_t n_v, const int32_t* __restrict__ F,
                                                   int64_t n, BuildState* __restrict__ st, uint64_t* __restrict__ keys,
                                                   uint32_t* __restrict__ vals) {
    __shared__ unsigned h[8][256];
    for (int d = 0; d < 8; d++) h[d][threadIdx.x] = 0u;
    __syncthreads();
    float ext = 0.0f;
    for (int a = 0; a < 3; a++) ext = fmaxf(ext, ord2f(st->hi[a]) - ord2f(st->lo[a]));
    const float qmax = 2097151.0f;
    const float sc = ext > 0.0f ? qmax / ext : 0.0f;
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < n; t += (int64_t)gridDim.x * kBlock) {
        float p[9];
        load_tri(V, n_v, F, t, p);
        uint32_t q[3];
        for (int a = 0; a < 3; a++)
            q[a] = (uint32_t)fminf(fmaxf((tri_centre(p, a) - ord2f(st->lo[a])) * sc, 0.0f), qmax);
        const uint64_t key = (spread21(q[0]) << 2) | (spread21(q[1]) << 1) | spread21(q[2]);
        keys[t] = key;
        vals[t] = (uint32_t)t;
        for (int d = 0; d < 8; d++) {
            // neighbours in the mesh often share the high digits: one addition then
            const unsigned digit = (unsigned)(key >> (8 * d)) & 255u;
            const unsigned one = __builtin_amdgcn_readfirstlane(digit);
            const unsigned long long same = __ballot(digit == one), act = __ballot(true);
            if (same == act) {
                if ((threadIdx.x & 63) == (unsigned)__builtin_ctzll(act)) atomicAdd(&h[d][one], (unsigned)__popcll(act));
            } else {
                atomicAdd(&h[d][digit], 1u);
            }
        }
    }
    __syncthreads();
    for (int d = 0; d < 8; d++) {
        const unsigned c = h[d][threadIdx.x];
        if (c) atomicAdd(&st->totals[d][threadIdx.x], c);
    }
}

// ---- sort of few triangles --------------------------------------------------
// One workgroup sorts up to kSortOne pairs in LDS by (code, triangle), a bitonic
// network: the radix sort's 24 launches take 116 us at any small size, this
// takes 28 us for the 1202 triangles of the city, 54 us for 3890.
constexpr int kSortOne = 4096, kSortBlock = 1024;
__global__ void __launch_bounds__(kSortBlock) k_sort_one(uint64_t* __restrict__ keys, uint32_t* __restrict__ vals, int n) {
    __shared__ uint64_t k[kSortOne];
    __shared__ uint32_t v[kSortOne];
    int size = 2;
    while (size < n) size *= 2;
    for (int i = threadIdx.x; i < size; i += kSortBlock) {
        k[i] = i < n ? keys[i] : ~0ull;
        v[i] = i < n ? vals[i] : 0xffffffffu;
    }
    __syncthreads();
    for (int run = 2; run <= size; run *= 2)
        for (int step = run / 2; step > 0; step /= 2) {
            for (int t = threadIdx.x; t < size / 2; t += kSortBlock) {
                const int i = 2 * t - (t & (step - 1)), j = i + step;
                const uint64_t a = k[i], b = k[j];
                const uint32_t x = v[i], y = v[j];
                const bool after = a > b || (a == b && x > y);
                if (after == ((i & run) == 0)) {
                    k[i] = b;
                    k[j] = a;
                    v[i] = y;
                    v[j] = x;
                }
            }
            __syncthreads();
        }
    for (int i = threadIdx.x; i < n; i += kSortBlock) {
        keys[i] = k[i];
        vals[i] = v[i];
    }
}

// ---- radix sort -----------------------------------------------------------
// A tile is kRsTile consecutive keys, kRsItems rounds of 64 per wavefront (8
// rather than 16 rounds fill the chip better: 1.76 -> 1.71 ms for a build of
// 1.02 M triangles and a first map).
// Digit counts of every tile, digit-major.
__global__ void __launch_bounds__(kBlock) k_rs_hist(const uint64_t* __restrict__ keys, int64_t n, int shift,
                                                    unsigned* __restrict__ hist, int ntiles) {
    __shared__ unsigned h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    int64_t base = (int64_t)blockIdx.x * kRsTile;
    for (int i = 0; i < kRsItems; i++) {
        int64_t idx = base + (int64_t)i * kBlock + threadIdx.x;
        if (idx < n) atomicAdd(&h[(keys[idx] >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[(int64_t)threadIdx.x * ntiles + blockIdx.x] = h[threadIdx.x];
}

// Turns digit d = blockIdx.x's counts into the first output index of every
// tile: the keys of smaller digits, then those of the tiles before.
__global__ void __launch_bounds__(kBlock) k_rs_offsets(unsigned* __restrict__ hist, int ntiles,
                                                       const unsigned* __restrict__ totals) {
    __shared__ unsigned part[kBlock];
    const int d = blockIdx.x, t = threadIdx.x;
    auto scan = [&](unsigned v) {      // inclusive over the block
        part[t] = v;
        __syncthreads();
        for (int off = 1; off < kBlock; off <<= 1) {
            const unsigned o = t >= off ? part[t - off] : 0u;
            __syncthreads();
            part[t] += o;
            __syncthreads();
        }
    };
    scan(t < d ? totals[t] : 0u);
    unsigned run = part[kBlock - 1];
    for (int b = 0; b < ntiles; b += kBlock) {
        unsigned* const h = hist + (int64_t)d * ntiles + b + t;
        const unsigned v = b + t < ntiles ? *h : 0u;
        __syncthreads();
        scan(v);
        if (b + t < ntiles) *h = run + part[t] - v;
        run += part[kBlock - 1];
    }
}

// Moves the keys of a tile to their places, in order.  A wavefront owns
// consecutive keys and its own running output index per digit, so that the
// rounds need no barrier: lanes with the same digit find each other with eight
// ballots, and the last of them advances the index (one index per block and
// five barriers a round: 20 us a pass over 1.02 M keys, 16 us so).
constexpr int kRsWaves = kBlock / 64;
__global__ void __launch_bounds__(kBlock) k_rs_scatter(const uint64_t* __restrict__ kin, const uint32_t* __restrict__ vin,
                                                       uint64_t* __restrict__ kout, uint32_t* __restrict__ vout, int64_t n,
                                                       int shift, const unsigned* __restrict__ offs, int ntiles) {
    __shared__ unsigned next[kRsWaves][256];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int w = 0; w < kRsWaves; w++) next[w][tid] = 0u;
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * kRsTile + (int64_t)wave * (kRsTile / kRsWaves) + lane;
    uint64_t key[kRsItems];
    uint32_t val[kRsItems];
#pragma unroll
    for (int r = 0; r < kRsItems; r++) {
        const int64_t idx = first + r * 64;
        key[r] = idx < n ? kin[idx] : 0ull;
        val[r] = idx < n ? vin[idx] : 0u;
        if (idx < n) atomicAdd(&next[wave][(key[r] >> shift) & 255u], 1u);
    }
    __syncthreads();
    // first output index of each wavefront's keys with digit tid
    unsigned run = offs[(int64_t)tid * ntiles + blockIdx.x];
    for (int w = 0; w < kRsWaves; w++) {
        const unsigned c = next[w][tid];
        next[w][tid] = run;
        run += c;
    }
    __syncthreads();
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
#pragma unroll
    for (int r = 0; r < kRsItems; r++) {
        const bool valid = first + r * 64 < n;
        const unsigned digit = (unsigned)(key[r] >> shift) & 255u;
        uint64_t m = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; b++) {
            const bool bit = (digit >> b) & 1u;
            const uint64_t bal = __ballot(bit);
            m &= bit ? bal : ~bal;
        }
        if (valid) {
            // every lane reads the index before the last one advances it: one
            // wavefront's LDS operations complete in order (volatile keeps them)
            volatile unsigned& idx = next[wave][digit];
            const unsigned at = idx + (unsigned)__popcll(m & lt);
            kout[at] = key[r];
            vout[at] = val[r];
            if ((m >> lane) == 1ull) idx = at + 1;
        }
    }
}

// ---- scan -----------------------------------------------------------------
// Exclusive scan of `count` unsigned values in place, one block of 1024
// (used for the per-tile sums of the multi-block scan below).
__global__ void k_scan1(unsigned* __restrict__ data, int64_t count) {
    __shared__ unsigned part[1024];
    const int T = 1024;
    int64_t per = (count + T - 1) / T;
    int64_t b = threadIdx.x * per, e = min(count, b + per);
    unsigned s = 0;
    for (int64_t i = b; i < e; i++) s += data[i];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < T; off <<= 1) {
        unsigned v = (threadIdx.x >= (unsigned)off) ? part[threadIdx.x - off] : 0u;
        __syncthreads();
        part[threadIdx.x] += v;
        __syncthreads();
    }
    unsigned run = part[threadIdx.x] - s;   // exclusive prefix of this chunk
    for (int64_t i = b; i < e; i++) {
        unsigned v = data[i];
        data[i] = run;
        run += v;
    }
}

// Multi-block exclusive scan: tiles of kScanTile values, one 256-thread block
// each.  Pass 1 writes every tile's sum, the sums are scanned by k_scan1, and
// pass 2 scans each tile from its offset.  A tile is staged in LDS with one
// pad word per 32 so that a thread's 16 consecutive values sit in distinct
// banks.
constexpr int kScanTile = 4096;
constexpr int kScanPer = kScanTile / kBlock;

__device__ __forceinline__ int scan_pad(int j) { return j + (j >> 5); }

__global__ void __launch_bounds__(kBlock) k_scan_sums(const unsigned* __restrict__ data, int64_t count,
                                                      unsigned* __restrict__ sums) {
    __shared__ unsigned red[kBlock];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    unsigned s = 0;
    for (int i = 0; i < kScanPer; i++) {
        const int64_t idx = base + (int64_t)i * kBlock + threadIdx.x;
        if (idx < count) s += data[idx];
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int off = kBlock / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = red[0];
}

__global__ void __launch_bounds__(kBlock) k_scan_tiles(const unsigned* data, unsigned* out, int64_t count,
                                                       const unsigned* __restrict__ offs) {
    __shared__ unsigned tile[kScanTile + kScanTile / 32];
    __shared__ unsigned part[kBlock];
    const int t = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    for (int i = 0; i < kScanPer; i++) {
        const int j = i * kBlock + t;
        tile[scan_pad(j)] = base + j < count ? data[base + j] : 0u;
    }
    __syncthreads();
    unsigned s = 0;
    for (int i = 0; i < kScanPer; i++) s += tile[scan_pad(t * kScanPer + i)];
    part[t] = s;
    __syncthreads();
    for (int off = 1; off < kBlock; off <<= 1) {
        unsigned v = t >= off ? part[t - off] : 0u;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    unsigned run = offs[blockIdx.x] + part[t] - s;
    for (int i = 0; i < kScanPer; i++) {
        const int j = scan_pad(t * kScanPer + i);
        const unsigned v = tile[j];
        tile[j] = run;
        run += v;
    }
    __syncthreads();
    for (int i = 0; i < kScanPer; i++) {
        const int j = i * kBlock + t;
        if (base + j < count) out[base + j] = tile[scan_pad(j)];
    }
}

// ---- gather ---------------------------------------------------------------
// Triangles in slot order with their AABBs: two float4 each, (lo.xyz, hi.x) and
// (hi.yz, -, -).
__global__ void k_gather(const float* __restrict__ V, int64_t n_v, const int32_t* __restrict__ F,
                         const uint32_t* __restrict__ order, const int32_t* __restrict__ M, int64_t n,
                         float4* __restrict__ tris, float4* __restrict__ normals, float4* __restrict__ boxes) {
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    int64_t t = order[s];
    float p[9];
    load_tri(V, n_v, F, t, p);
    int32_t m = M[t];
    tris[3 * s + 0] = make_float4(p[0], p[1], p[2], __int_as_float((int)t));
    tris[3 * s + 1] = make_float4(p[3], p[4], p[5], __int_as_float(m));
    tris[3 * s + 2] = make_float4(p[6], p[7], p[8], 0.0f);
    boxes[2 * s] = make_float4(tri_lo(p, 0), tri_lo(p, 1), tri_lo(p, 2), tri_hi(p, 0));
    boxes[2 * s + 1] = make_float4(tri_hi(p, 1), tri_hi(p, 2), 0.0f, 0.0f);
    double e1x = (double)p[3] - p[0], e1y = (double)p[4] - p[1], e1z = (double)p[5] - p[2];
    double e2x = (double)p[6] - p[0], e2y = (double)p[7] - p[1], e2z = (double)p[8] - p[2];
    double nx = e1y * e2z - e1z * e2y, ny = e1z * e2x - e1x * e2z, nz = e1x * e2y - e1y * e2x;
    double len = sqrt(nx * nx + ny * ny + nz * nz);
    if (len > 0.0) {
        nx /= len;
        ny /= len;
        nz /= len;
    } else {
        nx = 0.0;
        ny = 0.0;
        nz = 1.0;
    }
    normals[s] = make_float4((float)nx, (float)ny, (float)nz, __int_as_float(m));
}

// ---- boxes of runs of triangles -------------------------------------------
struct Box {
    float lo[3], hi[3];
};
__device__ __forceinline__ void box_add(Box& b, const float4* __restrict__ boxes, int64_t i) {
    const float4 p = boxes[2 * i], q = boxes[2 * i + 1];
    b.lo[0] = fminf(b.lo[0], p.x);
    b.lo[1] = fminf(b.lo[1], p.y);
    b.lo[2] = fminf(b.lo[2], p.z);
    b.hi[0] = fmaxf(b.hi[0], p.w);
    b.hi[1] = fmaxf(b.hi[1], q.x);
    b.hi[2] = fmaxf(b.hi[2], q.y);
}
__device__ __forceinline__ void box_store(float4* __restrict__ boxes, int64_t i, const Box& b) {
    boxes[2 * i] = make_float4(b.lo[0], b.lo[1], b.lo[2], b.hi[0]);
    boxes[2 * i + 1] = make_float4(b.hi[1], b.hi[2], 0.0f, 0.0f);
}
constexpr Box kNoBox = {{INFINITY, INFINITY, INFINITY}, {-INFINITY, -INFINITY, -INFINITY}};

// Levels follow one another in `boxes`, each holding the union of every 16
// entries of the level before it.  One launch makes three: a block turns 4096
// entries at `in` into 256, 16 and 1.
__global__ void __launch_bounds__(kBlock) k_box_levels(float4* __restrict__ boxes, int64_t in, int64_t count) {
    __shared__ float4 sh[2 * kBlock];
    const int64_t c1 = (count + 15) / 16, c2 = (c1 + 15) / 16, c3 = (c2 + 15) / 16;
    const int64_t out1 = in + count, out2 = out1 + c1, out3 = out2 + c2;
    const int t = threadIdx.x;
    const int64_t i1 = (int64_t)blockIdx.x * kBlock + t;
    Box b = kNoBox;
    for (int64_t i = 16 * i1; i < min(count, 16 * i1 + 16); i++) box_add(b, boxes, in + i);
    if (i1 < c1) box_store(boxes, out1 + i1, b);
    box_store(sh, t, b);
    __syncthreads();
    Box b2 = kNoBox;
    if (t < 16) {
        for (int i = 0; i < 16; i++) box_add(b2, sh, 16 * t + i);
        const int64_t i2 = (int64_t)blockIdx.x * 16 + t;
        if (i2 < c2) box_store(boxes, out2 + i2, b2);
    }
    __syncthreads();
    if (t < 16) box_store(sh, t, b2);
    __syncthreads();
    if (t == 0 && (int64_t)blockIdx.x < c3) {
        Box b3 = kNoBox;
        for (int i = 0; i < 16; i++) box_add(b3, sh, i);
        box_store(boxes, out3 + blockIdx.x, b3);
    }
}

// Union of the boxes of slots [a, b]: single entries up to the next multiple of
// 16 on both sides, then the level above, until few are left.
__device__ __forceinline__ Box box_range(const float4* __restrict__ boxes, int64_t n, int levels, int64_t a, int64_t b) {
    Box r = kNoBox;
    int64_t off = 0, cnt = n;
    for (int l = 0;; l++) {
        if (b - a < 32 || l == levels) {
            for (int64_t i = a; i <= b; i++) box_add(r, boxes, off + i);
            return r;
        }
        while (a & 15) box_add(r, boxes, off + a++);
        while ((b + 1) & 15) box_add(r, boxes, off + b--);
        a >>= 4;
        b = ((b + 1) >> 4) - 1;
        off += cnt;
        cnt = (cnt + 15) / 16;
    }
}

// ---- hierarchy ------------------------------------------------------------
__device__ __forceinline__ int lcp(const uint64_t* __restrict__ k, int64_t n, int64_t i, int64_t j) {
    if (j < 0 || j >= n) return -1;
    uint64_t a = k[i], b = k[j];
    if (a == b) return 64 + __clz((unsigned)(i ^ j));
    return __clzll(a ^ b);
}

__global__ void k_hierarchy(const uint64_t* __restrict__ keys, int64_t n, const float4* __restrict__ boxes, int levels,
                            float4* __restrict__ nodes) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n - 1) return;
    int d = (lcp(keys, n, i, i + 1) - lcp(keys, n, i, i - 1)) >= 0 ? 1 : -1;
    int dmin = lcp(keys, n, i, i - d);
    int64_t lmax = 2;
    while (lcp(keys, n, i, i + lmax * d) > dmin) lmax *= 2;
    int64_t l = 0;
    for (int64_t t = lmax / 2; t >= 1; t /= 2)
        if (lcp(keys, n, i, i + (l + t) * d) > dmin) l += t;
    int64_t j = i + l * d;
    int dnode = lcp(keys, n, i, j);
    int64_t s = 0, t = l;
    do {
        t = (t + 1) >> 1;
        if (lcp(keys, n, i, i + (s + t) * d) > dnode) s += t;
    } while (t > 1);
    const int64_t g = i + s * d + min(d, 0);
    const int64_t first = min(i, j), end = max(i, j);
    const int left = first == g ? ~(int)g : (int)g;
    const int right = end == g + 1 ? ~(int)(g + 1) : (int)(g + 1);
    const Box L = box_range(boxes, n, levels, first, g), R = box_range(boxes, n, levels, g + 1, end);
    nodes[4 * i + 0] = make_float4(L.lo[0], L.hi[0], L.lo[1], L.hi[1]);
    nodes[4 * i + 1] = make_float4(R.lo[0], R.hi[0], R.lo[1], R.hi[1]);
    nodes[4 * i + 2] = make_float4(L.lo[2], L.hi[2], R.lo[2], R.hi[2]);
    nodes[4 * i + 3] = make_float4(__int_as_float(left), __int_as_float(right), 0.0f, 0.0f);
}

// ---- 4-wide collapse -------------------------------------------------------
// A wide node is rooted at a binary node; its children are obtained by
// repeatedly replacing the internal child with the largest box surface area by
// its two children, until there are four children or only leaves.
__device__ __forceinline__ int2 node_refs(const float4* __restrict__ nodes, int i) {
    const float4 q = nodes[4 * (int64_t)i + 3];
    return make_int2(__float_as_int(q.x), __float_as_int(q.y));
}

__device__ __forceinline__ void node_box(const float4* __restrict__ nodes, int c, float lo[3], float hi[3]) {
    float4 q0 = nodes[4 * (int64_t)c], q1 = nodes[4 * (int64_t)c + 1], q2 = nodes[4 * (int64_t)c + 2];
    lo[0] = fminf(q0.x, q1.x);
    hi[0] = fmaxf(q0.y, q1.y);
    lo[1] = fminf(q0.z, q1.z);
    hi[1] = fmaxf(q0.w, q1.w);
    lo[2] = fminf(q2.x, q2.z);
    hi[2] = fmaxf(q2.y, q2.w);
}

__device__ __forceinline__ float box_area(const float lo[3], const float hi[3]) {
    float dx = hi[0] - lo[0], dy = hi[1] - lo[1], dz = hi[2] - lo[2];
    return dx * dy + dy * dz + dz * dx;
}

// `depth`: depth of node i on entry of each child in dep.
__device__ __forceinline__ int wide_children(const float4* __restrict__ nodes, int i, int depth, int refs[4],
                                             int dep[4]) {
    const int2 c = node_refs(nodes, i);
    refs[0] = c.x;
    refs[1] = c.y;
    dep[0] = dep[1] = depth + 1;
    float area[4] = {-1.0f, -1.0f, -1.0f, -1.0f};
    auto measure = [&](int j) {
        area[j] = -1.0f;
        if (refs[j] >= 0) {
            float lo[3], hi[3];
            node_box(nodes, refs[j], lo, hi);
            area[j] = box_area(lo, hi);
        }
    };
    measure(0);
    measure(1);
    int cnt = 2;
    while (cnt < 4) {
        int best = -1;
        float bestA = -1.0f;
        for (int j = 0; j < cnt; j++)
            if (refs[j] >= 0 && area[j] > bestA) {
                bestA = area[j];
                best = j;
            }
        if (best < 0) break;
        const int2 g = node_refs(nodes, refs[best]);
        refs[best] = g.x;
        refs[cnt] = g.y;
        dep[best]++;
        dep[cnt] = dep[best];
        if (++cnt < 4) {
            measure(best);
            measure(cnt - 1);
        }
    }
    return cnt;
}

// ---- small scenes: a tree of least surface area ----------------------------
// Up to kSahMax triangles, the wide nodes are taken from a second binary tree,
// split top-down at the least expected cost (surface area times triangles on
// both sides, MacDonald and Booth 1990).  Codes put a triangle where its centre
// is, so that one as large as the scene (a ground plane) widens every box down
// to a single house's: on the city (1202 triangles, ground of 2) a segment
// visits 7.5 wide nodes of the Karras tree and 5.0 of this one.  Maps of 1e6 and
// 1e7 rays 162 -> 135 and 618 -> 539 us, 64 rooftop transmitters 6.3 -> 5.3 ms;
// in the build k_sah_top takes 127 and k_sah_small 59 us.  The line at 4096 is
// what one workgroup makes in reasonable time, not where the tree stops to gain:
// boxes on a ground of 4,334, 5,810 and 8,114 triangles would build in 802, 904 and
// 1036 us instead of 396, 399 and 407 and trace maps of 1e6 rays in 379, 162 and
// 190 us instead of 406, 216 and 245 (1e7: 1.74, 0.93, 0.98 ms instead of 2.15, 1.16,
// 1.24), so that a scene kept for some ten such maps would gain.  The 1.02
// M-triangle terrain, whose triangles are alike, would be visited 9 % less.
//
// Node numbers are those of a depth-first walk: the left child of node i is
// i + 1, the right one i + (leaves on the left); triangle order within a node
// is kept by every split.  So the tree does not depend on the order in which
// its parts are made.
constexpr int kSahMax = 4096;
constexpr int kSahBins = 16, kSahSmall = 64;
constexpr int kSahBlock = 1024, kSahWaves = kSahBlock / 64;
constexpr int kSahDeep = 32;               // at this depth and below, halves
constexpr int kSahQueue = kSahMax / kSahSmall;

__device__ __forceinline__ void wave_fence() {
    __threadfence_block();
    __builtin_amdgcn_wave_barrier();
}
// These two round the same wherever they are inlined (no contraction): a count
// and the partition that it sizes must agree.
__device__ __forceinline__ float box_centre(const Box& b, int a) {
#pragma clang fp contract(off)
    return 0.5f * b.lo[a] + 0.5f * b.hi[a];
}
__device__ __forceinline__ int sah_bin(float centre, float lo, float scale) {
#pragma clang fp contract(off)
    return (int)fminf((centre - lo) * scale, (float)(kSahBins - 1));
}
__device__ __forceinline__ void box_add_if(Box& to, const Box& b, bool on) {
    for (int x = 0; x < 3; x++) {
        to.lo[x] = fminf(to.lo[x], on ? b.lo[x] : INFINITY);
        to.hi[x] = fmaxf(to.hi[x], on ? b.hi[x] : -INFINITY);
    }
}
// A triangle's box with its slot, as box_store writes it but for the slot.
struct SahBox {
    Box box;
    int id;
};
__device__ __forceinline__ SahBox sah_load(const float4* __restrict__ p, int i) {
    const float4 u = p[2 * i], v = p[2 * i + 1];
    return SahBox{{{u.x, u.y, u.z}, {u.w, v.x, v.y}}, __float_as_int(v.z)};
}
__device__ __forceinline__ void sah_store(float4* __restrict__ p, int i, const SahBox& b) {
    p[2 * i] = make_float4(b.box.lo[0], b.box.lo[1], b.box.lo[2], b.box.hi[0]);
    p[2 * i + 1] = make_float4(b.box.hi[1], b.box.hi[2], __int_as_float(b.id), 0.0f);
}
// Four loads in flight: f(box, index, index < end) for the wavefront's indices
// lo + lane, in order.
template <typename F>
__device__ __forceinline__ void sah_for(const float4* __restrict__ p, int lo, int end, int lane, F f) {
    for (int i = lo + lane; i - lane < end; i += 256) {
        SahBox b[4];
#pragma unroll
        for (int k = 0; k < 4; k++) b[k] = sah_load(p, min(i + 64 * k, end - 1));
#pragma unroll
        for (int k = 0; k < 4; k++)
            if (i - lane + 64 * k < end) f(b[k], i + 64 * k, i + 64 * k < end);
    }
}
// FLT_MAX at most, so that an overflow still orders; no box: 0
__device__ __forceinline__ float split_cost(const Box& l, int nl, const Box& r, int nr) {
    return fminf(box_area(l.lo, l.hi) * (float)nl + box_area(r.lo, r.hi) * (float)nr, FLT_MAX);
}
__device__ __forceinline__ void node_store(float4* __restrict__ nodes, int i, const Box& L, const Box& R, int left,
                                           int right) {
    nodes[4 * (int64_t)i + 0] = make_float4(L.lo[0], L.hi[0], L.lo[1], L.hi[1]);
    nodes[4 * (int64_t)i + 1] = make_float4(R.lo[0], R.hi[0], R.lo[1], R.hi[1]);
    nodes[4 * (int64_t)i + 2] = make_float4(L.lo[2], L.hi[2], R.lo[2], R.hi[2]);
    nodes[4 * (int64_t)i + 3] = make_float4(__int_as_float(left), __int_as_float(right), 0.0f, 0.0f);
}

// Least and greatest of a wavefront's values, on every lane: data-parallel
// primitives (rows of 16 by shifts, then across the rows).
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_or(float v, float none) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(none), __float_as_int(v), CTRL, ROWS, 0xf, false));
}
template <typename F>
__device__ __forceinline__ float wave_fold(float v, float none, F f) {
    v = f(v, dpp_or<0x111, 0xf>(v, none));
    v = f(v, dpp_or<0x112, 0xf>(v, none));
    v = f(v, dpp_or<0x114, 0xf>(v, none));
    v = f(v, dpp_or<0x118, 0xf>(v, none));
    v = f(v, dpp_or<0x142, 0xa>(v, none));
    v = f(v, dpp_or<0x143, 0xc>(v, none));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ void wave_union(Box& b) {
    for (int x = 0; x < 3; x++) {
        b.lo[x] = wave_fold(b.lo[x], INFINITY, [](float p, float q) { return fminf(p, q); });
        b.hi[x] = wave_fold(b.hi[x], -INFINITY, [](float p, float q) { return fmaxf(p, q); });
    }
}

// Splits every node of more than kSahSmall triangles, level by level: bounds of
// the centres, kSahBins bins per axis, the best of the 3 (kSahBins - 1) planes
// (one per lane), a stable partition.  A node's triangles are shared out over
// wavefronts that a level of few nodes leaves idle, each of which chooses the
// same plane from the common bins.  A level takes 12 us (bound by latency: four
// rounds of loads, as many barriers) to 35 (the bins' LDS atomics, on which all
// wavefronts wait): 266 us on 3890 triangles, 189 on 2354 and 127 on 1202; with
// one wavefront per node, sums by LDS permutes and every extreme an atomic 375,
// 231 and 136.  A task is {first, end, node, -}; those left for k_sah_small are
// {first, end, node, which of the two buffers}.  At the end, the depth of the
// Karras tree `karras`, by doubling the parent links.
__global__ void __launch_bounds__(kSahBlock) k_sah_top(const float4* __restrict__ boxes, int n,
                                                       const float4* __restrict__ karras, float4* __restrict__ nodes,
                                                       float4* buf0, float4* buf1, int4* __restrict__ small,
                                                       BuildState* __restrict__ st) {
    __shared__ unsigned bins[kSahWaves][3][kSahBins][7];     // ordered-int lo, hi; count
    __shared__ float part[kSahWaves][12];                    // a wavefront's bounds, then its boxes of both halves
    __shared__ int n_lefts[kSahWaves];
    __shared__ int4 list[2][kSahQueue];
    __shared__ int count[2], largest[2], n_small;        // of a level's nodes: number, most triangles
    __shared__ unsigned short par[kSahMax], dep[kSahMax];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < n; i += kSahBlock) {
        SahBox b = sah_load(boxes, i);
        b.id = i;
        sah_store(buf0, i, b);
    }
    if (threadIdx.x == 0) {
        n_small = n <= kSahSmall ? 1 : 0;
        count[0] = 1 - n_small;
        count[1] = 0;
        largest[0] = n;
        largest[1] = 0;
        if (n_small) small[0] = make_int4(0, n, 0, 0);
        else list[0][0] = make_int4(0, n, 0, 0);
    }
    __syncthreads();
    for (int level = 0; count[level & 1] > 0; level++) {
        const float4* in = level & 1 ? buf1 : buf0;
        float4* out = level & 1 ? buf0 : buf1;
        const int n_tasks = count[level & 1];
        // wavefronts per node: 256 triangles are one round of loads for one
        int g = kSahWaves;
        while (g > 1 && (n_tasks * g > kSahWaves || largest[level & 1] <= 128 * g)) g >>= 1;
        // the same number of rounds and barriers for every wavefront
        auto sync = [&]() {
            if (g > 1) {
                __threadfence_block();
                __syncthreads();
            } else {
                wave_fence();
            }
        };
        const int sub = wave & (g - 1), lead = wave - sub;
        for (int t0 = 0; t0 < n_tasks; t0 += kSahWaves / g) {
            const bool has = t0 + wave / g < n_tasks;
            const int4 task = list[level & 1][has ? t0 + wave / g : 0];
            const int lo = task.x, hi = task.y, cnt = hi - lo;
            // this wavefront's triangles (none without a node)
            const int each = ((cnt + g - 1) / g + 63) & ~63;
            const int s0 = has ? min(hi, lo + sub * each) : lo, s1 = has ? min(hi, s0 + each) : lo;
            unsigned(*const bn)[kSahBins][7] = bins[lead];
            if (sub == 0)
                for (int i = lane; i < 3 * kSahBins * 7; i += 64) (&bn[0][0][0])[i] = i % 7 < 3 ? 0xffffffffu : 0u;
            Box c = kNoBox;
            sah_for(in, s0, s1, lane, [&](const SahBox& b, int, bool) {      // the last one again is no harm
                for (int a = 0; a < 3; a++) {
                    c.lo[a] = fminf(c.lo[a], box_centre(b.box, a));
                    c.hi[a] = fmaxf(c.hi[a], box_centre(b.box, a));
                }
            });
            wave_union(c);
            if (lane == 0)
                for (int a = 0; a < 3; a++) {
                    part[wave][a] = c.lo[a];
                    part[wave][3 + a] = c.hi[a];
                }
            sync();
            float scale[3];
            for (int a = 0; a < 3; a++) {
                for (int w = lead; w < lead + g; w++) {
                    c.lo[a] = fminf(c.lo[a], part[w][a]);
                    c.hi[a] = fmaxf(c.hi[a], part[w][3 + a]);
                }
                const float ext = c.hi[a] - c.lo[a];
                scale[a] = ext > 0.0f ? (float)kSahBins / ext : 0.0f;
            }
            auto bin = [&](const Box& b, int a) { return sah_bin(box_centre(b, a), c.lo[a], scale[a]); };
            sah_for(in, s0, s1, lane, [&](const SahBox& b, int, bool on) {
                if (!on) return;
                // extremes first read: seldom does one move after the first few, and
                // reads at one address are one, atomics one per lane
                unsigned* w[3];
                unsigned now[3][6], own[6];
                for (int x = 0; x < 3; x++) {
                    own[x] = f2ord(b.box.lo[x]);
                    own[3 + x] = f2ord(b.box.hi[x]);
                }
                for (int a = 0; a < 3; a++) {
                    w[a] = bn[a][bin(b.box, a)];
                    for (int x = 0; x < 6; x++) now[a][x] = w[a][x];
                }
                for (int a = 0; a < 3; a++) {
                    atomicAdd(w[a] + 6, 1u);
                    for (int x = 0; x < 3; x++) {
                        if (own[x] < now[a][x]) atomicMin(w[a] + x, own[x]);
                        if (own[3 + x] > now[a][3 + x]) atomicMax(w[a] + 3 + x, own[3 + x]);
                    }
                }
            });
            sync();
            // lane = axis (kSahBins - 1) + plane
            const int axis = lane < kSahBins - 1 ? 0 : lane < 2 * (kSahBins - 1) ? 1 : 2;
            const int plane = lane - axis * (kSahBins - 1) + 1;
            Box L = kNoBox, R = kNoBox;
            int nl = 0, nr = 0;
            // (an empty bin's bounds read as NaN, which no minimum or maximum takes)
#pragma unroll 8
            for (int k = 0; k < kSahBins; k++) {
                const unsigned* const w = bn[axis][k];
                Box b;
                for (int x = 0; x < 3; x++) {
                    b.lo[x] = ord2f(w[x]);
                    b.hi[x] = ord2f(w[3 + x]);
                }
                box_add_if(L, b, k < plane);
                box_add_if(R, b, k >= plane);
                nl += k < plane ? (int)w[6] : 0;
                nr += k < plane ? 0 : (int)w[6];
            }
            float cost = plane < kSahBins && nl > 0 && nr > 0 ? split_cost(L, nl, R, nr) : INFINITY;
            // the first lane of the least cost
            const float least = wave_fold(cost, INFINITY, [](float p, float q) { return fminf(p, q); });
            const int best = __builtin_ctzll(__ballot(cost == least));
            const bool halves = !(least < INFINITY) || level >= kSahDeep;
            const int ax = __shfl(axis, best), pl = __shfl(plane, best);
            const int n_left = halves ? cnt / 2 : __shfl(nl, best);
            auto goes_left = [&](const SahBox& b, int i) {
                const int side = ax == 0 ? bin(b.box, 0) : ax == 1 ? bin(b.box, 1) : bin(b.box, 2);
                return halves ? i < lo + n_left : side < pl;
            };
            // those that go left before this wavefront's first
            int done_l = 0;
            if (g > 1) {
                int mine = 0;
                sah_for(in, s0, s1, lane, [&](const SahBox& b, int i, bool on) {
                    mine += (int)__popcll(__ballot(on && goes_left(b, i)));
                });
                if (lane == 0) n_lefts[wave] = mine;
                sync();
                for (int w = lead; w < wave; w++) done_l += n_lefts[w];
            }
            int done_r = s0 - lo - done_l;
            L = R = kNoBox;
            sah_for(in, s0, s1, lane, [&](const SahBox& b, int i, bool on) {
                const bool left = on && goes_left(b, i);
                const unsigned long long ml = __ballot(left), mr = __ballot(on && !left);
                const unsigned long long below = (1ull << lane) - 1ull;
                box_add_if(L, b.box, left);
                box_add_if(R, b.box, on && !left);
                if (on)
                    sah_store(out, left ? lo + done_l + (int)__popcll(ml & below)
                                        : lo + n_left + done_r + (int)__popcll(mr & below), b);
                done_l += (int)__popcll(ml);
                done_r += (int)__popcll(mr);
            });
            wave_union(L);
            wave_union(R);
            if (lane == 0)
                for (int x = 0; x < 3; x++) {
                    part[wave][x] = L.lo[x];
                    part[wave][3 + x] = L.hi[x];
                    part[wave][6 + x] = R.lo[x];
                    part[wave][9 + x] = R.hi[x];
                }
            sync();
            if (has && sub == 0 && lane == 0) {
                for (int w = lead + 1; w < lead + g; w++)
                    for (int x = 0; x < 3; x++) {
                        L.lo[x] = fminf(L.lo[x], part[w][x]);
                        L.hi[x] = fmaxf(L.hi[x], part[w][3 + x]);
                        R.lo[x] = fminf(R.lo[x], part[w][6 + x]);
                        R.hi[x] = fmaxf(R.hi[x], part[w][9 + x]);
                    }
                const int mid = lo + n_left, node = task.z;
                const int4 child[2] = {make_int4(lo, mid, node + 1, (level + 1) & 1),
                                       make_int4(mid, hi, node + n_left, (level + 1) & 1)};
                int ref[2];
                for (int k = 0; k < 2; k++) {
                    const int size = child[k].y - child[k].x;
                    ref[k] = size == 1 ? ~sah_load(out, child[k].x).id : child[k].z;
                    if (size > kSahSmall) {
                        list[(level + 1) & 1][atomicAdd(&count[(level + 1) & 1], 1)] = child[k];
                        atomicMax(&largest[(level + 1) & 1], size);
                    }
                    if (size > 1 && size <= kSahSmall) small[atomicAdd(&n_small, 1)] = child[k];
                }
                node_store(nodes, node, L, R, ref[0], ref[1]);
            }
            sync();      // `part` and the bins are free again
        }
        __threadfence_block();
        __syncthreads();
        if (threadIdx.x == 0) count[level & 1] = largest[level & 1] = 0;
        __syncthreads();
    }
    // depth of the Karras tree: dep = links followed so far, par = where they lead
    const int n_int = n - 1;
    for (int i = threadIdx.x; i < n_int; i += kSahBlock) dep[i] = i > 0 ? 1 : 0;
    if (threadIdx.x == 0) par[0] = 0;
    for (int i = threadIdx.x; i < n_int; i += kSahBlock) {
        const int2 r = node_refs(karras, i);
        if (r.x >= 0) par[r.x] = (unsigned short)i;
        if (r.y >= 0) par[r.y] = (unsigned short)i;
    }
    __syncthreads();
    constexpr int kEach = kSahMax / kSahBlock;
    int deepest = 0;
    for (int step = 1; step < n_int; step *= 2) {
        unsigned short p2[kEach], d2[kEach];
        for (int k = 0; k < kEach; k++) {
            const int i = threadIdx.x + k * kSahBlock;
            if (i < n_int) {
                p2[k] = par[par[i]];
                d2[k] = dep[i] + dep[par[i]];
            }
        }
        __syncthreads();
        for (int k = 0; k < kEach; k++) {
            const int i = threadIdx.x + k * kSahBlock;
            if (i < n_int) {
                par[i] = p2[k];
                dep[i] = d2[k];
            }
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < n_int; i += kSahBlock) deepest = max(deepest, (int)dep[i] + 1);
    for (int off = 32; off >= 1; off >>= 1) deepest = max(deepest, __shfl_xor(deepest, off));
    if (lane == 0) atomicMax(&st->max_depth, deepest);
    if (threadIdx.x == 0) st->n_small = n_small;
}

// One wavefront per subtree of at most kSahSmall triangles, one triangle per
// lane, all nodes of a level at once: a node's triangles are the lanes [s, e),
// each tries the plane at its own centre on the three axes, and the cheapest
// sorts them in two.
constexpr int kSmallBlock = 256;
__global__ void __launch_bounds__(kSmallBlock) k_sah_small(float4* __restrict__ nodes,
                                                           const float4* __restrict__ buf0, const float4* __restrict__ buf1,
                                                           const int4* __restrict__ small,
                                                           const BuildState* __restrict__ st) {
    struct Lane {
        Box box[64];
        int id[64];
        float cost[64];
        int axis[64], left[64];
    };
    __shared__ Lane sh[kSmallBlock / 64];
    const int lane = threadIdx.x & 63;
    Lane& w = sh[threadIdx.x >> 6];
    const int n_small = st->n_small;
    for (int t = blockIdx.x * (kSmallBlock / 64) + (threadIdx.x >> 6); t < n_small; t += gridDim.x * (kSmallBlock / 64)) {
        const int4 task = small[t];
        const int m = task.y - task.x;
        int s = lane < m ? 0 : lane, e = lane < m ? m : lane, node = task.z;
        const SahBox own = sah_load(task.w ? buf1 : buf0, task.x + min(lane, m - 1));
        int id = own.id;
        Box b = own.box;
        while (__ballot(e - s > 1)) {
            w.box[lane] = b;
            wave_fence();
            float key[3];
            for (int a = 0; a < 3; a++) key[a] = box_centre(b, a);
            Box L[3] = {kNoBox, kNoBox, kNoBox}, R[3] = {kNoBox, kNoBox, kNoBox};
            int nl[3] = {0, 0, 0};
            for (int j = s; j < e; j++) {
                const Box o = w.box[j];
                for (int a = 0; a < 3; a++) {
                    const float k = box_centre(o, a);
                    const bool left = k < key[a] || (k == key[a] && j <= lane);
                    box_add_if(L[a], o, left);
                    box_add_if(R[a], o, !left);
                    nl[a] += left ? 1 : 0;
                }
            }
            float cost = INFINITY;
            int axis = 0, mine = 0;
            Box bl = kNoBox, br = kNoBox;
#pragma unroll
            for (int a = 0; a < 3; a++) {
                const float c = nl[a] < e - s ? split_cost(L[a], nl[a], R[a], e - s - nl[a]) : INFINITY;
                const bool take = c < cost;
                cost = take ? c : cost;
                axis = take ? a : axis;
                mine = take ? nl[a] : mine;
                for (int x = 0; x < 3; x++) {
                    bl.lo[x] = take ? L[a].lo[x] : bl.lo[x];
                    bl.hi[x] = take ? L[a].hi[x] : bl.hi[x];
                    br.lo[x] = take ? R[a].lo[x] : br.lo[x];
                    br.hi[x] = take ? R[a].hi[x] : br.hi[x];
                }
            }
            w.cost[lane] = cost;
            w.axis[lane] = axis;
            w.left[lane] = mine;
            wave_fence();
            // every lane has a plane that parts its node, but for the last centre of
            // each axis, so a node of two or more always has a finite cost
            int win = s;
            float least = w.cost[s];
#pragma unroll 4
            for (int j = s + 1; j < e; j++) {
                const float c = w.cost[j];
                win = c < least ? j : win;
                least = c < least ? c : least;
            }
            const bool split = e - s > 1;
            const int n_left = split ? w.left[win] : 0, ax = split ? w.axis[win] : 0;
            const Box wb = w.box[split ? win : lane];
            const float kw = ax == 0 ? box_centre(wb, 0) : ax == 1 ? box_centre(wb, 1) : box_centre(wb, 2);
            const float k = ax == 0 ? key[0] : ax == 1 ? key[1] : key[2];
            const bool left = split && (k < kw || (k == kw && lane <= win));
            const unsigned long long ml = __ballot(left), mr = __ballot(split && !left);
            const unsigned long long below = (1ull << lane) - (1ull << s);       // lanes [s, lane)
            const int at = !split ? lane : left ? s + (int)__popcll(ml & below) : s + n_left + (int)__popcll(mr & below);
            const bool winner = split && lane == win;
            wave_fence();
            w.box[at] = b;
            w.id[at] = id;
            wave_fence();
            b = w.box[lane];
            id = w.id[lane];
            if (winner)
                node_store(nodes, node, bl, br, n_left == 1 ? ~w.id[s] : node + 1,
                           e - s - n_left == 1 ? ~w.id[s + n_left] : node + n_left);
            if (split) {
                if (lane < s + n_left) {
                    e = s + n_left;
                    node = node + 1;
                } else {
                    s = s + n_left;
                    node = node + n_left;
                }
            }
            wave_fence();
        }
    }
}

// One level of wide nodes, entries {node, depth} of `cur`: marks their internal
// children and appends them to `next` (one atomic on *total per block and
// round; `total` may lie in LDS).  Every thread of the block calls it.
__device__ __forceinline__ void wide_level(const float4* __restrict__ nodes, const int2* __restrict__ cur, int count,
                                           int2* __restrict__ next, int* total, unsigned* __restrict__ flags,
                                           int first, int step, int& deepest) {
    __shared__ int sh_n, sh_base;
    for (int e0 = first; e0 < count; e0 += step) {
        const int e = e0 + threadIdx.x;
        int refs[4], dep[4], cnt = 0, mine = 0, at = 0;
        if (threadIdx.x == 0) sh_n = 0;
        __syncthreads();
        if (e < count) {
            const int2 nd = cur[e];
            cnt = wide_children(nodes, nd.x, nd.y, refs, dep);
            for (int j = 0; j < cnt; j++) {
                if (refs[j] >= 0) mine++;
                else deepest = max(deepest, dep[j]);
            }
            if (mine) at = atomicAdd(&sh_n, mine);
        }
        __syncthreads();
        if (threadIdx.x == 0) sh_base = sh_n ? atomicAdd(total, sh_n) : 0;
        __syncthreads();
        at += sh_base;
        for (int j = 0; j < cnt; j++)
            if (refs[j] >= 0) {
                flags[refs[j]] = 1u;
                next[at++] = make_int2(refs[j], dep[j]);
            }
    }
}

__device__ __forceinline__ void report_depth(int deepest, BuildState* __restrict__ st, bool wanted) {
    if (!wanted) return;
    for (int off = 32; off >= 1; off >>= 1) deepest = max(deepest, __shfl_xor(deepest, off));
    if ((threadIdx.x & 63) == 0 && deepest > 0) atomicMax(&st->max_depth, deepest);
}

// The first levels, one block after another's barrier instead of a launch each,
// until a level has more than `most` nodes.  Level l's list is
// lists + (l & 1) n_int.
constexpr int kTopBlock = 1024;
__global__ void __launch_bounds__(kTopBlock) k_wide_top(const float4* __restrict__ nodes, int64_t n_int,
                                                        int most, int2* lists, unsigned* __restrict__ flags,
                                                        BuildState* __restrict__ st, bool depth) {
    __shared__ int n_next;
    int deepest = 0, count = 1, level = 0;
    if (threadIdx.x == 0) {
        lists[0] = make_int2(0, 0);
        flags[0] = 1u;
        st->count[0] = 1;
    }
    while (count > 0 && count <= most && level < kMaxLevels) {
        if (threadIdx.x == 0) n_next = 0;
        __threadfence_block();
        __syncthreads();
        wide_level(nodes, lists + (level & 1) * n_int, count, lists + ((level + 1) & 1) * n_int, &n_next, flags, 0,
                   kTopBlock, deepest);
        __threadfence_block();
        __syncthreads();
        count = n_next;
        level++;
        if (threadIdx.x == 0) st->count[level] = count;
        __syncthreads();
    }
    if (threadIdx.x == 0) st->next_level = level;
    report_depth(deepest, st, depth);
}

__global__ void __launch_bounds__(kBlock) k_wide_level(const float4* __restrict__ nodes, int64_t n_int, int level,
                                                       int2* lists, unsigned* __restrict__ flags,
                                                       BuildState* __restrict__ st, bool depth) {
    if (level < st->next_level) return;
    const int count = st->count[level];
    int deepest = 0;
    wide_level(nodes, lists + (level & 1) * n_int, count, lists + ((level + 1) & 1) * n_int, &st->count[level + 1], flags,
               blockIdx.x * kBlock, gridDim.x * kBlock, deepest);
    report_depth(deepest, st, depth);
}

// Writes the wide nodes numbered below `cap` and the number of all of them.
__global__ void k_wide_emit(const float4* __restrict__ nodes, const float4* __restrict__ tris,
                            const unsigned* __restrict__ is_root, const unsigned* __restrict__ index4, int64_t n_int,
                            int64_t cap, float4* __restrict__ wide, BuildState* __restrict__ st) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_int) return;
    if (i == n_int - 1) st->n_wide = index4[i] + is_root[i];
    if (!is_root[i] || (int64_t)index4[i] >= cap) return;
    int refs[4], dep[4];
    int cnt = wide_children(nodes, (int)i, 0, refs, dep);
    float lo[4][3], hi[4][3];
    int out[4];
    for (int j = 0; j < 4; j++) {
        if (j >= cnt) {
            // inverted box: no ray ever enters it
            for (int a = 0; a < 3; a++) {
                lo[j][a] = INFINITY;
                hi[j][a] = -INFINITY;
            }
            out[j] = RT_WIDE_EMPTY;
        } else if (refs[j] < 0) {
            int64_t sl = ~refs[j];
            float4 a0 = tris[3 * sl], a1 = tris[3 * sl + 1], a2 = tris[3 * sl + 2];
            lo[j][0] = fminf(fminf(a0.x, a1.x), a2.x);
            lo[j][1] = fminf(fminf(a0.y, a1.y), a2.y);
            lo[j][2] = fminf(fminf(a0.z, a1.z), a2.z);
            hi[j][0] = fmaxf(fmaxf(a0.x, a1.x), a2.x);
            hi[j][1] = fmaxf(fmaxf(a0.y, a1.y), a2.y);
            hi[j][2] = fmaxf(fmaxf(a0.z, a1.z), a2.z);
            out[j] = refs[j];
        } else {
            node_box(nodes, refs[j], lo[j], hi[j]);
            out[j] = (int)index4[refs[j]];
        }
    }
    float4* w = wide + 8 * (int64_t)index4[i];
    for (int a = 0; a < 3; a++) {
        w[2 * a] = make_float4(lo[0][a], lo[1][a], lo[2][a], lo[3][a]);
        w[2 * a + 1] = make_float4(hi[0][a], hi[1][a], hi[2][a], hi[3][a]);
    }
    w[6] = make_float4(__int_as_float(out[0]), __int_as_float(out[1]), __int_as_float(out[2]),
                       __int_as_float(out[3]));
    const int leaf = (out[0] < 0 ? 2 : 0) | (out[1] < 0 ? 4 : 0) | (out[2] < 0 ? 8 : 0) | (out[3] < 0 ? 16 : 0);
    w[7] = make_float4(__int_as_float(leaf), 0.0f, 0.0f, 0.0f);
}

inline unsigned grid_for(int64_t n, int block) { return (unsigned)std::max<int64_t>(1, (n + block - 1) / block); }

}  // namespace

// Tile sums needed by scan_exclusive for `count` values.
static int64_t scan_sums_len(int64_t count) { return (count + kScanTile - 1) / kScanTile; }

// Exclusive scan of `count` values of `data` into `out` (which may be data);
// `sums` holds scan_sums_len(count) values of scratch.
static void scan_exclusive(const unsigned* data, unsigned* out, int64_t count, unsigned* sums, hipStream_t st) {
    const int64_t tiles = scan_sums_len(count);
    if (tiles <= 0) return;
    hipLaunchKernelGGL(k_scan_sums, dim3((unsigned)tiles), dim3(kBlock), 0, st, data, count, sums);
    hipLaunchKernelGGL(k_scan1, dim3(1), dim3(1024), 0, st, sums, tiles);
    hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)tiles), dim3(kBlock), 0, st, data, out, count, sums);
}

// Histogram buffer of the radix sort for n keys: 256 digit counts per tile (it
// also holds the tile sums of a scan of n values).
static int64_t rs_hist_len(int64_t n) { return 256 * ((n + kRsTile - 1) / kRsTile); }

// Stack entries beyond the LDS part that a traversal of n triangles is expected
// to need at most: three per level of a 4-wide tree some levels deeper than a
// balanced one.
static int64_t expected_spill(int64_t n) {
    int bits = 1;
    while (((int64_t)1 << bits) < n) bits++;
    return std::max<int64_t>(0, 3 * (bits / 2 + 6) + 2 - RT_STACK_LDS);
}

// The traversal's spill area: at the end of the scene's allocation if it was
// made large enough, else one of its own.
rt_status rt_size_spill(rt_scene* s, void* spare, size_t spare_bytes) {
    const int64_t lanes = (int64_t)rt_persistent_blocks(64, s->device) * 64;
    s->spill_entries = (size_t)(std::max<int64_t>(0, rt_stack_need(s) - RT_STACK_LDS) * lanes);
    const size_t need = sizeof(int) * s->spill_entries;
    if (need <= spare_bytes) {
        s->spill = (int*)spare;
        return RT_OK;
    }
    hipError_t e = hipMalloc(&s->spill_own, need);
    if (e != hipSuccess) return rt_hip_fail(e, "hipMalloc(spill)");
    s->spill = (int*)s->spill_own;
    s->bytes += need;
    return RT_OK;
}

rt_status rt_build_lbvh(rt_scene* s, const float* V, int64_t n_v, const int32_t* F, const int32_t* M,
                        hipStream_t st) {
    const int64_t n = s->n_tri, n_int = std::max<int64_t>(0, n - 1);
    // one allocation: counters, nodes, triangles, normals, codes; the build's
    // flags and numbers; the wide nodes, or before them the sort and the box
    // levels (the level lists reuse the sort's part); the spill area
    size_t total = 0;
    auto part = [&](size_t bytes) {
        const size_t at = total;
        total += (bytes + 255) & ~(size_t)255;
        return at;
    };
    const size_t o_counters = part(sizeof(unsigned long long) * (RT_QUEUES + 1) * RT_QUEUE_STRIDE);
    const size_t o_nodes = part(sizeof(float4) * 4 * n_int);
    const size_t o_tris = part(sizeof(float4) * 3 * n);
    const size_t o_normals = part(sizeof(float4) * n);
    const size_t o_keys = part(sizeof(uint64_t) * n);
    const size_t o_state = part(sizeof(BuildState));
    const size_t o_flags = part(sizeof(unsigned) * n_int), o_index = part(sizeof(unsigned) * n_int);
    const bool sah = n >= 2 && n <= kSahMax;
    const size_t o_sah = part(sah ? sizeof(float4) * 4 * n_int : 0), o_buf = part(sah ? 2 * sizeof(float4) * 2 * n : 0),
                 o_small = part(sah ? sizeof(int4) * (n / 2) : 0);
    const size_t o_wide = total;
    const size_t o_k1 = part(sizeof(uint64_t) * n), o_v0 = part(sizeof(uint32_t) * n), o_v1 = part(sizeof(uint32_t) * n);
    const size_t o_hist = part(sizeof(unsigned) * (size_t)rs_hist_len(n));
    int64_t n_boxes = n;
    int levels = 0;
    for (int64_t c = n; c > 32;)
        for (int k = 0; k < 3; k++) {
            c = (c + 15) / 16;
            n_boxes += c;
            levels++;
        }
    const size_t o_boxes = part(sizeof(float4) * 2 * n_boxes);
    const size_t wide_node = sizeof(float4) * 8;
    // trees measured have 0.5 to 0.6 wide nodes per triangle
    total = std::max(total, o_wide + wide_node * (size_t)(n_int * 2 / 3 + 1));
    const size_t wide_bytes = total - o_wide;
    const size_t o_spill = part(n > 0 ? sizeof(int) * (size_t)expected_spill(n) * (size_t)rt_persistent_blocks(64, s->device) * 64
                                      : 0);
    hipError_t he = hipMalloc(&s->block, total);
    if (he != hipSuccess) return rt_hip_fail(he, "rt_build_scene: hipMalloc");
    s->bytes = total;
    char* const base = (char*)s->block;
    s->counters = (unsigned long long*)(base + o_counters);
    if (n == 0) {
        s->root = -1;
        s->depth = 0;
        return rt_size_spill(s, base + o_spill, total - o_spill);
    }
    s->nodes = (float4*)(base + o_nodes);
    s->tris = (float4*)(base + o_tris);
    s->normals = (float4*)(base + o_normals);
    s->morton = (uint64_t*)(base + o_keys);
    BuildState* const state = (BuildState*)(base + o_state);
    unsigned *const flags = (unsigned*)(base + o_flags), *const index4 = (unsigned*)(base + o_index);
    uint64_t *ka = s->morton, *kb = (uint64_t*)(base + o_k1);
    uint32_t *va = (uint32_t*)(base + o_v0), *vb = (uint32_t*)(base + o_v1);
    unsigned* const hist = (unsigned*)(base + o_hist);
    float4* const boxes = (float4*)(base + o_boxes);
    int2* const lists = (int2*)(base + o_k1);
    const float4* const tree = sah ? (float4*)(base + o_sah) : s->nodes;      // what the wide nodes are made of

    hipEvent_t e0 = nullptr, e1 = nullptr;
    auto cleanup = [&]() {
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
    };
    HIPCHK(hipEventCreate(&e0));
    HIPCHK(hipEventCreate(&e1));
    HIPCHK(hipEventRecord(e0, st));
    const unsigned g = grid_for(n, kBlock);
    hipLaunchKernelGGL(k_build_init, dim3(std::min(g, 1024u)), dim3(kBlock), 0, st, state, flags, n_int);
    hipLaunchKernelGGL(k_bounds, dim3(std::min(g, 512u)), dim3(kBlock), 0, st, V, n_v, F, M, s->n_mat, n, state);
    hipLaunchKernelGGL(k_morton, dim3(std::min(g, 512u)), dim3(kBlock), 0, st, V, n_v, F, n, state, ka, va);
    const int rs_blocks = (int)((n + kRsTile - 1) / kRsTile);
    if (n <= kSortOne) hipLaunchKernelGGL(k_sort_one, dim3(1), dim3(kSortBlock), 0, st, ka, va, (int)n);
    for (int shift = 0; shift < 64 && n > kSortOne; shift += 8) {
        const unsigned* const totals = state->totals[shift / 8];      // an address on the device
        hipLaunchKernelGGL(k_rs_hist, dim3(rs_blocks), dim3(kBlock), 0, st, ka, n, shift, hist, rs_blocks);
        hipLaunchKernelGGL(k_rs_offsets, dim3(256), dim3(kBlock), 0, st, hist, rs_blocks, totals);
        hipLaunchKernelGGL(k_rs_scatter, dim3(rs_blocks), dim3(kBlock), 0, st, ka, va, kb, vb, n, shift, hist,
                           rs_blocks);
        std::swap(ka, kb);
        std::swap(va, vb);
    }
    // after 8 passes (or none) the sorted data is back in (morton, v0)
    hipLaunchKernelGGL(k_gather, dim3(g), dim3(kBlock), 0, st, V, n_v, F, va, M, n, s->tris, s->normals, boxes);
    constexpr int kLevelBatch = 16, kTopLevels = 5;      // k_wide_top takes levels 0..4 at least (4^5 nodes)
    // no level of so few triangles has more nodes than k_wide_top takes (each holds
    // two triangles at least), and up to 4096 triangles two per thread cost less than
    // the launches (16, 71 us)
    const int most = n <= 4 * kTopBlock ? 2 * kTopBlock : kTopBlock;
    int level = n <= 2 * most ? kMaxLevels : kTopLevels;
    int64_t wide_cap = (int64_t)(wide_bytes / wide_node);
    auto queue_levels = [&]() {
        const unsigned gl = std::min(g, 512u);
        for (int k = 0; k < kLevelBatch && level < kMaxLevels; k++, level++)
            hipLaunchKernelGGL(k_wide_level, dim3(gl), dim3(kBlock), 0, st, tree, n_int, level, lists, flags, state, !sah);
    };
    auto queue_emit = [&](float4* wide, int64_t cap) {
        scan_exclusive(flags, index4, n_int, hist, st);
        hipLaunchKernelGGL(k_wide_emit, dim3(g), dim3(kBlock), 0, st, tree, s->tris, flags, index4, n_int, cap, wide,
                           state);
    };
    if (n_int > 0) {
        int64_t off = 0, c = n;
        for (int l = 0; l < levels; l += 3) {
            hipLaunchKernelGGL(k_box_levels, dim3((unsigned)((c + 4095) / 4096)), dim3(kBlock), 0, st, boxes, off, c);
            for (int k = 0; k < 3; k++) {
                off += c;
                c = (c + 15) / 16;
            }
        }
        hipLaunchKernelGGL(k_hierarchy, dim3(g), dim3(kBlock), 0, st, ka, n, boxes, levels, s->nodes);
        if (sah) {
            float4* const buf = (float4*)(base + o_buf);
            int4* const small = (int4*)(base + o_small);
            hipLaunchKernelGGL(k_sah_top, dim3(1), dim3(kSahBlock), 0, st, boxes, (int)n, s->nodes, (float4*)tree, buf,
                               buf + 2 * n, small, state);
            hipLaunchKernelGGL(k_sah_small, dim3((unsigned)std::min<int64_t>(256, (n + 31) / 32)), dim3(kSmallBlock), 0, st,
                               (float4*)tree, buf, buf + 2 * n, small, state);
        }
        hipLaunchKernelGGL(k_wide_top, dim3(1), dim3(kTopBlock), 0, st, tree, n_int, most, lists, flags, state, !sah);
        queue_levels();
        queue_emit((float4*)(base + o_wide), wide_cap);
    }
    HIPCHK(hipGetLastError());
    HIPCHK(hipEventRecord(e1, st));
    BuildState h;
    const size_t read_back = offsetof(BuildState, totals);
    HIPCHK(hipMemcpyAsync(&h, state, read_back, hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    if (h.err != 0) {
        cleanup();
        std::string why;
        if (h.err & 1u) why += " vertex index out of range;";
        if (h.err & 2u) why += " material id out of range;";
        if (h.err & 4u) why += " non-finite vertex coordinate;";
        return rt_fail(RT_EINVAL, "rt_build_scene: invalid mesh:" + why);
    }
    if (n_int > 0) {
        // a tree deeper than the queued levels (its lists are whole, but the
        // nodes were written over them): the levels again from the start
        while (h.count[std::min(level, kMaxLevels)] != 0) {
            if (level >= kMaxLevels) {
                cleanup();
                return rt_fail(RT_EDEVICE, "rt_build_scene: LBVH hierarchy is malformed");
            }
            const int upto = level + kLevelBatch;
            hipLaunchKernelGGL(k_build_init, dim3(std::min(g, 1024u)), dim3(kBlock), 0, st, state, flags, n_int);
            hipLaunchKernelGGL(k_wide_top, dim3(1), dim3(kTopBlock), 0, st, tree, n_int, most, lists, flags, state, !sah);
            level = kTopLevels;
            while (level < std::min(upto, kMaxLevels)) queue_levels();
            queue_emit((float4*)(base + o_wide), wide_cap);
            const BuildState first = h;
            HIPCHK(hipGetLastError());
            HIPCHK(hipMemcpyAsync(&h, state, read_back, hipMemcpyDeviceToHost, st));
            HIPCHK(hipStreamSynchronize(st));
            for (int a = 0; a < 3; a++) {
                h.lo[a] = first.lo[a];
                h.hi[a] = first.hi[a];
            }
            if (sah) h.max_depth = first.max_depth;
        }
        s->root = 0;
        s->depth = h.max_depth;
        while (s->wide_levels < kMaxLevels && h.count[s->wide_levels] > 0) s->wide_levels++;
        // the traversal addresses wide nodes with 32-bit byte offsets; larger
        // trees are traversed as binary trees
        const int64_t n4 = (int64_t)h.n_wide;
        if (n4 < ((int64_t)1 << 25)) {
            s->wide = (float4*)(base + o_wide);
            if (n4 > wide_cap) {
                HIPCHK(hipMalloc(&s->wide_own, wide_node * (size_t)n4));
                s->wide = (float4*)s->wide_own;
                s->bytes += wide_node * (size_t)n4;
                queue_emit(s->wide, n4);
                HIPCHK(hipGetLastError());
                HIPCHK(hipStreamSynchronize(st));
            }
            s->n_wide = n4;
        }
    } else {
        s->root = ~0;   // single triangle: the root is a leaf
    }
    float ms = 0.0f;
    HIPCHK(hipEventElapsedTime(&ms, e0, e1));
    s->build_ms = ms;
    for (int a = 0; a < 3; a++) {
        s->lo[a] = ord2f_host(h.lo[a]);
        s->hi[a] = ord2f_host(h.hi[a]);
    }
    cleanup();
    return rt_size_spill(s, base + o_spill, total - o_spill);
}
