// sbr_forward.hip -- persistent SBR radio-map kernel for gfx950.
//
// One lane carries one ray at a time.  A lane whose ray has ended takes the
// next lattice index from a device work queue (one atomic per wavefront,
// shared out with ballot/mbcnt), so wavefronts stay full while ray lengths
// differ (queue_entry says what a claim holds).  Per traced segment l the lane
//   1. finds the closest hit through the LBVH, the wavefront's lanes together
//      while they want the same nodes, else each on its own (short LDS stack,
//      spill to a per-lane global area sized from the tree depth), or by
//      testing every triangle when accel = brute force (validation);
//   2. deposits ||T C_T||^2 * lambda^2 / (4 pi N_S |M_i| |k_z|) into the plane
//      cell it crosses, if any (estimator eq. radio-map-solver-ci-all-2-
//      estimator for specular chains), either with one FP32 atomic or after
//      summing same-cell crossings across the wavefront;
//   3. unless the segment escaped or l = L, reflects specularly and updates
//      the 2x2 field transfer matrix T (eq. fresnel_vac and the bases of
//      eq. fresnel_in_vectors / eq. fresnel_out_vectors), or, where nothing
//      needs T, the field T C_T itself.
// The extended variant (template flag EXT) adds, per hit, the single-layer
// slab coefficients, the sampled interaction type (specular or diffuse
// reflection, transmission) with its 1/sqrt(q) weight, and early
// termination by Russian roulette or gain thresholding before the next
// segment; its random draws come from a counter-based Philox4x32-10 stream.
// Ray state (origin, direction, basis, T or field) stays in VGPRs for the whole
// ray.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstring>

#include "sbr_common.h"

using namespace rtd;

namespace {

struct FwdArgs {
    const float4* nodes;
    const float4* wide;
    const float4* tris;
    const float4* normals;
    int root;
    int n_tri;
    int n_wide;              // 4-wide nodes (0 when the tree is binary only)
    const float* eps_r;
    const float* sigma;
    TxDesc tx;
    PlaneDesc pl;
    int64_t ray_begin;
    int64_t n_work;
    int L;
    float t_min;
    int deposit;       // 1 atomic, 2 wave
    int npol;
    float* map;
    int64_t map_stride;
    float4* tape_seg;
    int* tape_nseg;
    int64_t tape_n;
    int32_t* hits;
    int32_t* cells;
    float* weights;
    unsigned long long* stats;
    // work queues (see queue_entry)
    unsigned long long* counter;   // RT_QUEUES heads, then the mask of drained queues, RT_QUEUE_STRIDE apart
    unsigned long long per_queue;  // entries per queue
    int64_t n_units;               // units of `claim` indices (`once`: of `width`)
    int64_t mid;                   // unit that comes first, -1 = in ascending order
    int nq;                        // queues in use (1..RT_QUEUES)
    int once;                      // 1: every wavefront has at most one unit, its own
    int width;                     // rays a wavefront starts at once, on its first lanes
    int claim;                     // work indices per unit
    int first_width;               // width of a wavefront's first unit
    unsigned n_first;              // leading entries of a queue that hold the indices [hole, hole + hole_size),
    int64_t hole, hole_size;       // first_width each
    unsigned n_claim;              // then, units of `claim`; the rest are of `width`
    unsigned run, n_run;           // consecutive units per queue turn, among the first n_run entries
    // early termination (kernel variant EXT): before segments l >= rr_depth
    int rr_depth;
    float rr_p_max;                // Russian roulette, 0 = off
    float gain_threshold;          // gain thresholding, 0 = off
    unsigned seed;
    float gain_scale;              // lambda^2 / (16 pi^2): path gain = gain_scale ||E||^2 / r^2
    float inv_kappa;               // 1 / tx.kappa: |alpha|^2 = kap * inv_kappa
    // finite-thickness walls and refraction (kernel variant EXT)
    const float* thickness;        // slab thickness per material (m), or null
    const float* scattering;       // scattering coefficient S per material, or null (no diffuse)
    const float* xpd;              // cross-polarisation share K_x per material
    const float* pattern;          // [n_mat][4] scattering pattern, or null (Lambertian)
    int refraction;                // 1: sample reflection or transmission at every hit
    float k0;                      // 2 pi / lambda
    int* spill;
    int64_t spill_stride;
    int spill_depth;
    int tape_groups;         // float4 records per segment on the tape (4, or 2 = geometry only)
    int refill;              // refill a wavefront once this many lanes are idle
    // several transmitters (MODE_MULTI, MODE_GEOM): device tables
    const TxDesc* txs;       // ordered largest budget first
    const int64_t* prefix;   // [n_tx + 1] exclusive prefix of the budgets
    const int32_t* slots;    // output slot of each ordered transmitter
    int n_tx;
    int64_t slot_stride;     // floats between the maps of consecutive slots
    // unit of entry i = r run + k of queue q, i < n_run: r by_r + k by_k + q by_q (runs of units per queue and turn:
    // nq run, 1 and run; or `run` stretches per queue in turn: 1, and nq and 1 times their length).  Down here:
    // further up these took the others off the boundaries that wide scalar loads need (0.5 %)
    unsigned by_r, by_k, by_q;
};

// Kernel modes: one transmitter; several transmitters with one material set
// (deposits into per-transmitter maps); several transmitters, geometry only
// (records hit slots, cells, directions and bases for a later field pass).
enum { MODE_SINGLE = 0, MODE_MULTI = 1, MODE_GEOM = 2 };

// Wavefront deposit: same-cell groups summed before the atomics (4 measured
// best against 1, 2 and no limit on the Manhattan and rooftop workloads).
constexpr int kDepositGroups = 4;

// Index of the transmitter whose ray range holds global ray g.
__device__ __forceinline__ int find_tx(const int64_t* __restrict__ prefix, int n_tx, int64_t g) {
    int lo = 0, hi = n_tx;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (prefix[mid] <= g) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Work of entry i of queue q: indices [*first, *end), possibly none.
//
// The grid is what is resident (four wavefronts per SIMD); each wavefront
// starts with the entry of its number and claims the next from its queue's
// head with one atomic.  A wavefront of near-horizontal rays takes 0.13 ms in
// the city and 0.3 ms and more on the 1.02 M-triangle scene, as long as
// hundreds of others, so what counts in a call of few units per wavefront is
// that those start first: the units of one transmitter follow outward from the
// lattice's equator, above and below in turn, and straight-down and
// straight-up rays, the shortest, make the tail.  All wavefronts advance along
// one front, cut over the queues by unit, so that no queue is drained much
// before another (contiguous ranges per queue leave the horizon's range to the
// end); `run` units in a row go to one queue, whose workgroups share an XCD's
// L2, about a quarter of the front's turn in all.  Several transmitters come
// largest budget first, in lattice order, and change to units of one wavefront
// for the last 32 per wavefront.
//
// Against contiguous ranges on up to 256 queues with two grids' worth of
// workgroups, on one tree: city map, 1e6 rays 224 -> 160 us, 2e6 271 -> 168, 4e6
// 376 -> 293, 1e7 762 -> 645 us, 3e7 1.79 -> 1.78 ms; 1.02 M triangles, 1e6 622
// -> 558 us, 4e6 885 -> 696, 6.4e7 6.77 -> 6.85 ms; 64 rooftop transmitters of
// up to 1e7 rays 6.61 -> 6.35 ms.  Units of four wavefronts already at the
// horizon cost 0.3 ms more in the city at 1e6 rays.
//
// One front also brings the deposits together in the few cells under it.  Where
// a wavefront does not sum them first (one atomic per crossing, or a launch in
// lattice order, whose wavefronts hold no neighbours), calls of four units per
// wavefront and more go through several stretches at once instead, one per
// queue and turn (against one front, and in brackets the contiguous ranges on 256
// queues; city: lattice order, 5e6 rays 1.66 -> 1.13 ms [1.22], 2e7 6.56 -> 4.45
// [4.51]; atomics, 2e6 0.53 -> 0.45 [0.48], 5e6 1.45 -> 1.20 [1.21], 2e7 6.09 ->
// 4.74 [5.28]; three transmitters of 3e6 rays 3.6 -> 1.9 [2.1] and 4.6 -> 3.1 [3.4]).
// Few stretches suffice in lattice order, where the 1.02 M-triangle scene would
// lose 10 % at 1.5e6 rays with 16; atomics take 16 (with 4 the city's 1.1e6 rays
// take 0.33 ms, with 16 0.27).
//
// Where the tree is larger than an L2 (4 MB) a fetch takes longer and so do
// the wavefronts at the horizon: in calls of up to six units per wavefront the
// first units, nearest the equator, are then of 16 rays (1.02 M triangles, 9e4
// rays 416 -> 378 us, 2e5 554 -> 397, 4e5 501 -> 376, 1e6 547 -> 477, 4e6 would
// take 8 % more; the city would at 1e6 rays too, its fetches being short).  On
// smaller trees it depends on the scene: boxes on a ground of 19,202 triangles would
// gain at 2e5 rays (208 -> 172 us) and lose at 1.4e6 (218 -> 272), 49,154
// likewise (183 -> 163, 218 -> 267), 20,000 loose triangles lose throughout (2e5
// 779 -> 944).  With a refill threshold of 48 or less the lanes left idle refill after
// one segment: 1e6 rays gain 8 instead of 10 %, 1.4e6 nothing instead of 5.
//
// Several transmitters on such a tree have their horizons one after another, the
// last near the call's end; in calls of up to 64 units per wavefront in all and
// 8 per transmitter four stretches per queue spread them (64 transmitters of 5e4
// rays 1.40 -> 1.10 ms, 16 of 3e5 1.50 -> 1.24; larger calls lose: 32 of up to
// 2e6 rays 6.4 -> 7.4, 3 of 3e6 1.67 -> 1.80).  Below
// four units per wavefront one stretch per queue does for four transmitters and
// more (8 of 1e5 599 -> 541 us, 16 of 5e4 594 -> 558, 4 of 7e4 512 -> 434; 2 of
// 3e5 would take 606 instead of 512).
__device__ __forceinline__ void queue_entry(const FwdArgs& a, unsigned i, int q, int64_t* first, int64_t* end) {
    *first = *end = 0;
    if (i < a.n_first) {
        *first = a.hole + ((int64_t)i * a.nq + q) * a.first_width;
        *end = *first + a.first_width;
        return;
    }
    i -= a.n_first;
    if (i < a.n_claim) {
        // units are numbered in 32 bits
        const unsigned n_units = (unsigned)a.n_units;
        const int mid = (int)a.mid;
        unsigned u = i * (unsigned)a.nq + (unsigned)q;
        if (i < a.n_run) {
            const unsigned r = i / a.run, k = i - r * a.run;
            u = r * a.by_r + k * a.by_k + (unsigned)q * a.by_q;
        }
        if (u >= n_units) return;
        if (mid >= 0) {
            // outward from mid: the two sides in turn, then the rest of the longer one
            const unsigned below = (unsigned)mid, above = n_units - below, both = 2u * min(below, above), v = u >> 1;
            u = u < both ? ((u & 1u) ? below + v : below - 1u - v) : (below > above ? n_units - 1u - u : u);
        }
        *first = (int64_t)u * a.claim;
        if (*first >= a.hole) *first += a.hole_size;
        *end = min(a.n_work, *first + a.claim);
    } else {
        const int64_t f = (int64_t)a.n_claim * a.nq * a.claim + ((int64_t)(i - a.n_claim) * a.nq + q) * a.width;
        if (f >= a.n_work) return;
        *first = f;
        *end = min(a.n_work, f + a.width);
    }
}

// A wavefront leaves the common walk once the visits that few lanes wanted add
// up to this many of its active lanes (2, 4, 8 and 16 measure within 0.5 % of
// each other on the city and the 1.02 M-triangle scene).
constexpr int kPacketWaste = 8;

// The kernel's argument block, with its address hidden from the optimiser:
// each part of the ray loop reads the arguments it needs through the scalar
// cache.  Without this the compiler loads all of them before the loop, runs
// out of scalar registers and keeps over a hundred in vector-register lanes.
__device__ __forceinline__ const FwdArgs& kernel_args() {
    uintptr_t p = (uintptr_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const FwdArgs*)(const __attribute__((address_space(4))) FwdArgs*)p;
}

// A pointer to what no kernel writes while this one runs, the same on every
// lane: reads go through the scalar cache.
template <typename T>
__device__ __forceinline__ const T* scalar_pointer(const T* p) {
    const uintptr_t u = (uintptr_t)uniform_u64((unsigned long long)(uintptr_t)p);
    return (const T*)(const __attribute__((address_space(4))) T*)u;
}

// Per-lane traversal stack: the first RT_STACK_LDS entries {node, entry
// distance} live in LDS, laid out [entry][lane] (8 bytes each, so a
// wavefront's pushes are contiguous); deeper entries (node only) go to a
// per-lane global spill area.  `top` is the LDS slot of entry sp while
// sp <= RT_STACK_LDS.
struct TravStack {
    int2* top;
    int stride;   // lanes per workgroup
    int sp;
    unsigned gtid;
};

__device__ __forceinline__ int& spill_slot(const FwdArgs& a, int sp, unsigned gtid) {
    return a.spill[(sp - RT_STACK_LDS) * a.spill_stride + gtid];
}

// Stores entry sp, beyond the LDS part, of a wavefront's stack; returns sp, or
// sp - 1 if there is no room (cannot happen: the area is sized from the tree
// depth).  Reads the arguments it needs: the callers seldom come here.
__device__ __forceinline__ int push_spill(int ref, int sp, unsigned gtid, unsigned& overflow) {
    const FwdArgs& a = kernel_args();
    if (sp - RT_STACK_LDS >= a.spill_depth) {
        overflow |= 1u;
        return sp - 1;
    }
    spill_slot(a, sp, gtid) = ref;
    return sp;
}

__device__ __forceinline__ void push_entry(const FwdArgs& a, TravStack& st, int ref, float key, unsigned& overflow) {
    if (st.sp < RT_STACK_LDS) {
        *st.top = make_int2(ref, __float_as_int(key));
        st.top += st.stride;
    } else if (st.sp - RT_STACK_LDS < a.spill_depth) {
        spill_slot(a, st.sp, st.gtid) = ref;
    } else {
        overflow |= 1u;   // cannot happen: the spill area is sized from the tree depth
        return;
    }
    st.sp++;
}

// Pop until an entry whose box may still hold a hit closer than `lim`.
__device__ __forceinline__ bool pop_entry(const FwdArgs& a, TravStack& st, float lim, int& node) {
    while (st.sp > 0) {
        st.sp--;
        if (st.sp < RT_STACK_LDS) {
            st.top -= st.stride;
            const int2 e = *st.top;
            if (__int_as_float(e.y) <= lim) {
                node = e.x;
                return true;
            }
        } else {
            node = spill_slot(a, st.sp, st.gtid);
            return true;
        }
    }
    return false;
}

// Best hit so far of one query: ties in t go to the smallest original id.
struct Best {
    float t, lim;     // distance; cull limit = t times the slack, kept finite (see closest_hit)
    int id, slot;
};

__device__ __forceinline__ void take_hit(Best& b, bool hit, float t, int id, int s) {
    const bool better = hit & ((t < b.t) | ((t == b.t) & (id < b.id)));
    b.t = better ? t : b.t;
    b.id = better ? id : b.id;
    b.slot = better ? s : b.slot;
    b.lim = better ? fminf(t * kBoxSlack, FLT_MAX) : b.lim;
}

// Set bits of a mask, counted and kept in scalar registers.
__device__ __forceinline__ int count_lanes(unsigned long long m) {
    int n;
    asm("s_bcnt1_i32_b64 %0, %1" : "=s"(n) : "s"(m) : "scc");
    return n;
}

// Value i (0..3, from its two lowest bits) of four.
template <typename T>
__device__ __forceinline__ T pick4(T v0, T v1, T v2, T v3, unsigned i) {
    const T a = (i & 1u) ? v1 : v0, b = (i & 1u) ? v3 : v2;
    return (i & 2u) ? b : a;
}

// First part of a 4-wide closest-hit query: the active lanes of the wavefront
// walk the tree together, one node at a time, for as long as enough of them
// want the same nodes.  Node planes and triangles are fetched once per
// wavefront through the scalar cache, so a visit costs 11 VALU instructions
// per child box and no vector memory access; a lane takes part with its own
// cull limit.  Deferred children go to the same per-lane stack that the
// per-lane loop uses (a lane that missed the child stores an INFINITY key, which
// never passes a cull), so the wavefront can leave for the per-lane loop
// after any node.  Returns false when the query is complete; else `node` is
// the node at which this lane has to go on, or -1 if it has to pop one.
//
// Why: the launch order makes a wavefront's rays neighbours, and a plane
// mirrors them together.  With 1e8 rays on the 1.02 M-triangle scene 61 of 64
// lanes are active per segment, and a common walk takes 11.5 node visits and
// 2.2 triangle tests per wavefront and segment where the per-lane loop takes
// 14.3 and 4.6; its node visit issues about 118 VALU instructions and returns
// 7 KiB through the vector memory path, both nearly saturated (93 % of the
// VALU cycles).  The walk is bound by instruction issue and by branches: the
// same walk with early exits in the triangle test and a branch per child and
// push took 13.6 ms where this form took 12.1 (15.2 without the walk); the
// city, 1e7 rays, 0.88, 0.80 and 0.95 ms (11.8 and 0.53 ms now, with the queues
// below, a better tree for the city and cheaper masks).
template <bool REC>
__device__ __forceinline__ bool packet_phase(const FwdArgs& a, const Ray& r, int last, float tmin, Best& best,
                                             int2* __restrict__ stk, int lstride, unsigned gtid, int& sp,
                                             unsigned& n_nodes, unsigned& n_tris, unsigned& overflow, int& node_out) {
    // the rays have to share the order of near and far planes and the axis
    // permutation of the triangle test
    const int nx = uniform((int)r.nx), ny = uniform((int)r.ny), nz = uniform((int)r.nz);
    const int kx = uniform(r.kx), ky = uniform(r.ky), kz = uniform(r.kz);
    const unsigned long long act = ballot(true);
    const int n_act = count_lanes(act);
    node_out = 0;
    if (ballot((int)r.nx == nx && (int)r.ny == ny && (int)r.nz == nz && r.kx == kx && r.kz == kz) != act) return true;
    const float ox = pick(r.ox, r.oy, r.oz, kx), oy = pick(r.ox, r.oy, r.oz, ky), oz = pick(r.ox, r.oy, r.oz, kz);
    const float4* const wide = a.wide;
    const float4* const tris = a.tris;
    const int n_wide = a.n_wide;
    int node = 0, waste = 0;
    bool mine = true;                  // this lane wants `node`
    for (int guard = 0; guard < n_wide; guard++) {
        if (REC) n_nodes += mine ? 1u : 0u;
        const WideNode w = load_node_uniform(wide, node, nx, ny, nz);
        float te[4];
        unsigned long long m[4];       // lanes that enter each child
#pragma unroll
        for (int c = 0; c < 4; c++) {
            te[c] = max3_raw(__builtin_fmaf(w.px[c], r.ix, r.cnx), __builtin_fmaf(w.py[c], r.iy, r.cny),
                             max_raw(__builtin_fmaf(w.pz[c], r.iz, r.cnz), tmin));
            const float f = min3_raw(__builtin_fmaf(w.qx[c], r.jx, r.cfx), __builtin_fmaf(w.qy[c], r.jy, r.cfy),
                                     min_raw(__builtin_fmaf(w.qz[c], r.jz, r.cfz), best.lim));
            m[c] = ballot(te[c] <= f);
        }
        // bit c + 1: some lane enters child c
        const unsigned hits = (m[0] ? 2u : 0u) | (m[1] ? 4u : 0u) | (m[2] ? 8u : 0u) | (m[3] ? 16u : 0u);
        unsigned leaves = hits & w.leaf, inner = hits & ~w.leaf;
        auto ref = [&](unsigned c) { return uniform(pick4(w.rf[0], w.rf[1], w.rf[2], w.rf[3], c)); };
        // entry distance of child c, INFINITY on lanes that miss it
        auto entry = [&](unsigned c) {
            const float e = pick4(te[0], te[1], te[2], te[3], c);
            return __builtin_amdgcn_inverse_ballot_w64(pick4(m[0], m[1], m[2], m[3], c)) ? e : INFINITY;
        };
        while (leaves) {
            const unsigned c = (unsigned)__builtin_ctz(leaves) - 1u;
            leaves &= leaves - 1u;
            const int s = ~ref(c);
            const bool want = (entry(c) <= best.lim) & (s != last);
            if (REC) n_tris += want ? 1u : 0u;
            float t;
            int id;
            const bool hit = tri_hit_axes(r, tris, s, kx, ky, kz, ox, oy, oz, tmin, t, id);
            take_hit(best, want & hit, t, id, s);
        }
        // internal children: the one that most lanes enter first is descended,
        // the others are deferred
        int next = -1;
        float key = INFINITY;
        if (inner) {
            unsigned c = (unsigned)__builtin_ctz(inner) - 1u;
            next = ref(c);
            key = entry(c);
            inner &= inner - 1u;
            while (inner) {
                c = (unsigned)__builtin_ctz(inner) - 1u;
                inner &= inner - 1u;
                const int r2 = ref(c);
                const float k2 = entry(c);
                const bool swap = count_lanes(ballot(k2 < key)) > count_lanes(ballot(key < k2));
                const int far_ref = swap ? next : r2;
                if (__builtin_expect(sp < RT_STACK_LDS, 1))
                    stk[sp * lstride] = make_int2(far_ref, __float_as_int(swap ? key : k2));
                else
                    sp = push_spill(far_ref, sp, gtid, overflow);
                sp++;
                next = swap ? r2 : next;
                key = swap ? k2 : key;
            }
        }
        mine = key <= best.lim;
        unsigned long long live = ballot(mine);
        while (live == 0ull) {
            if (sp == 0) return false;
            sp--;
            if (__builtin_expect(sp < RT_STACK_LDS, 1)) {
                const int2 e = stk[sp * lstride];
                next = uniform(e.x);
                mine = __int_as_float(e.y) <= best.lim;
            } else {
                next = uniform(spill_slot(kernel_args(), sp, gtid));
                mine = true;
            }
            live = ballot(mine);
        }
        node = next;
        if (__builtin_expect((unsigned)node >= (unsigned)n_wide, 0)) {
            overflow |= 1u;
            return false;
        }
        // a visit that fewer than a third of the lanes want costs more than
        // its share of the per-lane loop: leave after a few of them
        waste = max(0, waste + n_act - 3 * count_lanes(live));
        if (__builtin_expect(waste > kPacketWaste * n_act, 0)) {
            node_out = mine ? node : -1;
            return true;
        }
    }
    return false;
}

// Closest hit of ray r among all triangles but `last` (a slot).  Ties in t go
// to the smallest original triangle id.  best.slot = -1: none.
template <bool BRUTE, bool WIDE, bool REC>
__device__ __forceinline__ Best closest_hit(const FwdArgs& a, float3 o, float3 k, int last, int2* __restrict__ stk,
                                            int lstride, unsigned gtid, unsigned& n_nodes, unsigned& n_tris,
                                            unsigned& overflow) {
    // cull limit: t times the slack, kept finite so that the INFINITY keys of
    // missed, leaf and empty slots never pass it, also before the first hit;
    // updated with t
    Best best = {INFINITY, FLT_MAX, 0x7fffffff, -1};
    // canonical once, so that the min/max below need no per-use quieting
    const float tmin = __builtin_canonicalizef(a.t_min);
    if (a.n_tri == 0) return best;
    Ray r = make_ray(o, k);
    auto test = [&](int s) {
        if (s == last) return;
        float4 v0 = a.tris[3 * (int64_t)s], v1 = a.tris[3 * (int64_t)s + 1], v2 = a.tris[3 * (int64_t)s + 2];
        if (REC) n_tris++;
        float t;
        const bool hit = tri_hit(r, v0, v1, v2, tmin, t);
        take_hit(best, hit, t, __float_as_int(v0.w), s);
    };
    if (BRUTE) {
        for (int s = 0; s < a.n_tri; s++) test(s);
        return best;
    }
    if (a.root < 0) {
        test(~a.root);
        return best;
    }
    TravStack st{stk, lstride, 0, gtid};
    if (WIDE) {
        // 4-wide traversal: four slab tests per node fetch (empty child slots
        // hold inverted boxes and never hit); leaf children are tested at once,
        // internal hits are sorted by entry distance, the nearest is descended
        // and the others are pushed farthest first
        int node = 0;
        int sp = 0;
        if (!packet_phase<REC>(a, r, last, tmin, best, stk, lstride, gtid, sp, n_nodes, n_tris, overflow, node)) return best;
        st.sp = sp;
        st.top = stk + min(sp, RT_STACK_LDS) * lstride;
        if (node < 0 && !pop_entry(a, st, best.lim, node)) return best;
        // the ray's constants are made again (from hidden copies, so that they
        // are not the same values to the compiler): held across the loop above
        // they would cost its registers
        hide(o);
        hide(k);
        r = make_ray(o, k);
        const __amdgpu_buffer_rsrc_t rs = wide_rsrc(a.wide, a.n_wide);
        for (int guard = 0; guard < a.n_tri; guard++) {
            if (REC) n_nodes++;
            bool h[4];
            float te[4];
            int ref[4];
            box4(r, rs, (unsigned)node << 7, tmin, best.lim, h, te, ref);
            // keys of the internal hits: the entry distance's bits with the
            // child's index in the lowest two (distances are >= 0, so the bits
            // order like the numbers, and clearing two of them only brings a
            // child nearer); the others sort last and, as NaN, pass no cull
            unsigned key[4];
            unsigned leaves = 0;
#pragma unroll
            for (int c = 0; c < 4; c++) {
                key[c] = (h[c] && ref[c] >= 0) ? (__float_as_uint(te[c]) & ~3u) | (unsigned)c : 0xffffffffu;
                leaves |= (h[c] && ref[c] < 0) ? 1u << c : 0u;
            }
            // select by the bits of c (selects, not a branch per slot)
            auto child = [&](unsigned c) {
                return pick4(ref[0], ref[1], ref[2], ref[3], c);
            };
            // one triangle-test body for the whole wavefront: it runs as many
            // times as the lane with the most leaf hits needs
            while (leaves) {
                const unsigned c = (unsigned)__builtin_ctz(leaves);
                leaves &= leaves - 1u;
                test(~child(c));
            }
            // sorted: the least, middle and largest of the first three, then the
            // fourth between them
            const unsigned lo = min(min(key[0], key[1]), key[2]), hi = max(max(key[0], key[1]), key[2]);
            const unsigned mid = med3_u32(key[0], key[1], key[2]);
            const unsigned srt[4] = {min(lo, key[3]), med3_u32(lo, mid, key[3]), med3_u32(mid, hi, key[3]), max(hi, key[3])};
            // children entered beyond the closest hit so far are dropped (the
            // same outcome as a box test with the new bound)
            if (__uint_as_float(srt[0]) <= best.lim) {
                // seldom more than one child in any lane: one test then skips all
                // the pushes
                if (ballot(__uint_as_float(srt[1]) <= best.lim)) {
                    if (ballot(__uint_as_float(srt[2]) <= best.lim)) {
                        if (__uint_as_float(srt[3]) <= best.lim)
                            push_entry(a, st, child(srt[3]), __uint_as_float(srt[3]), overflow);
                        if (__uint_as_float(srt[2]) <= best.lim)
                            push_entry(a, st, child(srt[2]), __uint_as_float(srt[2]), overflow);
                    }
                    if (__uint_as_float(srt[1]) <= best.lim)
                        push_entry(a, st, child(srt[1]), __uint_as_float(srt[1]), overflow);
                }
                node = child(srt[0]);
            } else if (!pop_entry(a, st, best.lim, node)) {
                break;
            }
        }
        return best;
    }
    int node = a.root;
    // every internal node is visited at most once per query; the bound only
    // guards against a malformed tree
    for (int guard = 0; guard < a.n_tri; guard++) {
        if ((unsigned)node >= (unsigned)(a.n_tri - 1)) {
            overflow |= 1u;
            break;
        }
        if (REC) n_nodes++;
        const float4* q = a.nodes + 4 * (int64_t)node;
        float4 q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
        bool hL, hR;
        float tL, tR;
        box2(r, q0, q1, q2, tmin, best.t * kBoxSlack, hL, hR, tL, tR);
        int cl = __float_as_int(q3.x), cr = __float_as_int(q3.y);
        if (hL && cl < 0) {
            test(~cl);
            hL = false;
        }
        if (hR && cr < 0) {
            test(~cr);
            hR = false;
        }
        if (hL && hR) {
            // the far child's entry distance goes with it, so that it can be
            // dropped at pop time without fetching its node
            const bool lnear = tL <= tR;
            push_entry(a, st, lnear ? cr : cl, lnear ? tR : tL, overflow);
            node = lnear ? cl : cr;
        } else if (hL) {
            node = cl;
        } else if (hR) {
            node = cr;
        } else if (!pop_entry(a, st, best.t * kBoxSlack, node)) {
            break;
        }
    }
    return best;
}

// What a ray carries from segment to segment (template parameter FIELD):
//   0          the 2x2 transfer matrix T and the launch patterns C (E = T C),
//              which the tape stores and the extensions' decisions are made of;
//   1, 2       the fields E of one or two polarisations: half the registers and
//              arithmetic of T with one polarisation.
template <int FIELD>
struct FieldState {
    cf e[FIELD][2];
    __device__ __forceinline__ void set(int p, float ct, float cp) {
        e[p][0] = cf{ct, 0.0f};
        e[p][1] = cf{cp, 0.0f};
    }
    __device__ __forceinline__ void launch() {}
    __device__ __forceinline__ float power(int p) const { return cabs2(e[p][0]) + cabs2(e[p][1]); }
    // E <- diag(c_perp, -c_par) W E
    __device__ __forceinline__ void interact(const Bounce& b, cf cperp, cf cpar) {
        const cf mr = cf{-cpar.re, -cpar.im};
#pragma unroll
        for (int p = 0; p < FIELD; p++) {
            const cf u0 = cadd(cscale(e[p][0], b.w00), cscale(e[p][1], b.w01));
            const cf u1 = cadd(cscale(e[p][0], b.w10), cscale(e[p][1], b.w11));
            e[p][0] = cmul(cperp, u0);
            e[p][1] = cmul(mr, u1);
        }
    }
};

template <>
struct FieldState<0> {
    cf Ta, Tb, Tc, Td;
    float c0t, c0p, c1t, c1p;   // C_T per polarisation
    __device__ __forceinline__ void set(int p, float ct, float cp) {
        if (p == 0) {
            c0t = ct;
            c0p = cp;
        } else {
            c1t = ct;
            c1p = cp;
        }
    }
    __device__ __forceinline__ void launch() {
        Ta = cf{1, 0};
        Tb = cf{0, 0};
        Tc = cf{0, 0};
        Td = cf{1, 0};
    }
    __device__ __forceinline__ float power(int p) const {
        const float ct = p == 0 ? c0t : c1t, cp = p == 0 ? c0p : c1p;
        const cf e0 = cadd(cscale(Ta, ct), cscale(Tb, cp));
        const cf e1 = cadd(cscale(Tc, ct), cscale(Td, cp));
        return cabs2(e0) + cabs2(e1);
    }
    // T <- diag(c_perp, -c_par) W T: the new basis is (e_perp, k' x e_perp),
    // whose second vector is -e_par of the outgoing wave for both k' = k_r and
    // k' = k
    __device__ __forceinline__ void interact(const Bounce& b, cf cperp, cf cpar) {
        const cf na = cmix_exact(Ta, b.w00, Tc, b.w01), nb = cmix_exact(Tb, b.w00, Td, b.w01);
        const cf nc = cmix_exact(Ta, b.w10, Tc, b.w11), nd = cmix_exact(Tb, b.w10, Td, b.w11);
        const cf mr = cf{-cpar.re, -cpar.im};
        Ta = cmul_exact(cperp, na);
        Tb = cmul_exact(cperp, nb);
        Tc = cmul_exact(mr, nc);
        Td = cmul_exact(mr, nd);
    }
};

// REC: the call has records, statistics or a tape; FIELD: see FieldState (0
// with REC and EXT).
template <bool BRUTE, int MODE, bool WIDE, bool EXT, bool REC, int FIELD>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) k_forward(const FwdArgs) {
    extern __shared__ int2 s_stack[];
    const int lstride = blockDim.x;
    int2* stk = s_stack + threadIdx.x;
    const unsigned gtid = blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = (int)__lane_id();
    constexpr bool FIELDS = MODE != MODE_GEOM;
    constexpr bool TAPE = REC || MODE == MODE_GEOM;

    unsigned st_seg = 0, st_cross = 0, st_nodes = 0, st_tris = 0, st_over = 0;

    bool active = false;
    bool exhausted = false;
    // this wavefront's queue (a workgroup's wavefronts share one, and so do the
    // workgroups that share an XCD) and first entry
    int q = 0;
    int looks = 0;                     // at the mask of drained queues
    int width = kernel_args().first_width;
    int64_t res_b = 0, res_e = 0;      // claimed work indices, not yet started
    {
        const FwdArgs& a = kernel_args();
        const unsigned w = (unsigned)uniform((int)(threadIdx.x >> 6)), per_block = blockDim.x >> 6;
        exhausted = a.once != 0;
        if (a.once) {
            // neighbouring wavefronts from eight stretches of the order, so that the
            // long ones do not share a CU
            const int64_t each = (a.n_units + 7) >> 3, wave = (int64_t)blockIdx.x * per_block + w;
            if ((wave >> 3) < each) {
                res_b = min(a.n_work, ((wave & 7) * each + (wave >> 3)) * a.width);
                res_e = min(a.n_work, res_b + a.width);
            }
        } else {
            q = (int)(blockIdx.x % (unsigned)a.nq);
            queue_entry(a, blockIdx.x / (unsigned)a.nq * per_block + w, q, &res_b, &res_e);
        }
    }
    int64_t rid = 0;          // ray index relative to ray_begin
    int l = 0;
    int last = -1;
    float3 o = f3(0, 0, 0), k = f3(0, 0, 0), es = f3(0, 0, 0);
    FieldState<FIELDS ? FIELD : 0> fs;
    float kap = 0.0f;         // lambda^2 / (4 pi N_S |M|) of the lane's transmitter, times |alpha|^2
    float rlen = 0.0f;        // unfolded length to the last interaction (early termination only)
    // several transmitters: the map of the lane's transmitter, the lattice
    // index of its ray there (the counter of its random streams, as in a
    // single call), 1 / kappa and the output slot of that transmitter
    float* mapb = nullptr;
    int64_t nlat = 0;
    float ikap = 0.0f;
    int tslot = 0;
    int txi = 0;              // transmitter of the wavefront's last launch

    while (true) {
        // ---- refill lanes without a ray: from this wavefront's reservoir of
        // claimed work indices, claiming more when it cannot cover every idle
        // lane
        if (!exhausted || res_b < res_e) {
            const FwdArgs& a = kernel_args();
            const unsigned long long own = ~0ull >> (64 - width);
            const unsigned long long need = ballot(!active) & own;
            if (need && (__popcll(need) >= a.refill || need == own)) {
                const unsigned cnt = (unsigned)__popcll(need);
                // wave-uniform: every value below is the same on all lanes
                const int64_t b1 = res_b, e1 = res_e;
                int64_t b2 = 0, e2 = 0;
                while (e1 - b1 < (int64_t)cnt && b2 == e2 && !exhausted) {
                    unsigned long long i = 0;
                    if (lane == 0) i = atomicAdd(a.counter + q * RT_QUEUE_STRIDE, 1ull);
                    i = uniform_u64(i);
                    if (i < a.per_queue) {
                        // the last entry of a queue (one claim per queue) marks it
                        if (i + 1 == a.per_queue && lane == 0)
                            atomicOr(a.counter + RT_QUEUES * RT_QUEUE_STRIDE, 1ull << q);
                        queue_entry(a, (unsigned)i, q, &b2, &e2);
                    } else {
                        // drained: on to the next queue that is not marked
                        unsigned long long m = 0;
                        if (lane == 0)
                            m = __hip_atomic_load(a.counter + RT_QUEUES * RT_QUEUE_STRIDE, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
                        m = ~uniform_u64(m) & ((1ull << a.nq) - 1ull) & ~(1ull << q);
                        // a bound on the looks: every queue is emptied by its own
                        // wavefronts, so leaving early loses nothing
                        exhausted = m == 0ull || ++looks > 2 * RT_QUEUES;
                        const unsigned long long up = m >> q << q;
                        if (m) q = __builtin_ctzll(up ? up : m);
                    }
                }
                // idle lanes take the reservoir first, then the new batch
                const int64_t n1 = e1 - b1;
                const int64_t take1 = min((int64_t)cnt, n1);
                const int64_t take2 = min((int64_t)cnt - take1, e2 - b2);
                width = a.width;
                res_b = take1 < n1 ? b1 + take1 : b2 + take2;
                res_e = take1 < n1 ? e1 : e2;
                if (!active && lane < width) {
                    const unsigned rank = __builtin_amdgcn_mbcnt_hi((unsigned)(need >> 32),
                                                                    __builtin_amdgcn_mbcnt_lo((unsigned)need, 0u));
                    const bool mine = rank < (unsigned)(take1 + take2);
                    const int64_t my = rank < (unsigned)take1 ? b1 + rank : b2 + (rank - (unsigned)take1);
                    auto begin = [&](const TxDesc& td, int64_t n) {
                        Launch Lr = fib_launch(n, td.n_rays);
                        if (FIELDS) {
                            float ct, cp;
                            tx_pattern<float>(Lr, td, td.pol == 1 ? 1 : 0, ct, cp);
                            fs.set(0, ct, cp);
                            if (FIELD == 2 || (FIELD == 0 && a.npol == 2)) {
                                tx_pattern<float>(Lr, td, 1, ct, cp);
                                fs.set(1, ct, cp);
                            }
                            // a transmit array scales the ray's field by alpha
                            // and its weights by |alpha|^2
                            kap = td.kappa;
                            if (td.n_ant > 0) kap *= array_gain(Lr, td);
                        }
                        k = f3((float)Lr.kx, (float)Lr.ky, (float)Lr.kz);
                        es = f3((float)Lr.tx, (float)Lr.ty, (float)Lr.tz);
                        o = f3(td.pos[0], td.pos[1], td.pos[2]);
                        fs.launch();
                        l = 0;
                        rlen = 0.0f;
                        last = -1;
                        active = true;
                        if (REC) {
                            const int stride = a.L + 1;
                            if (a.hits) {
                                for (int j = 0; j < stride; j++) a.hits[rid * stride + j] = -2;
                            }
                            if (a.cells) {
                                for (int j = 0; j < stride; j++) a.cells[rid * stride + j] = -1;
                            }
                            if (a.weights) {
                                for (int j = 0; j < stride; j++) a.weights[rid * stride + j] = 0.0f;
                            }
                        }
                    };
                    if constexpr (MODE == MODE_SINGLE) {
                        if (mine) {
                            rid = launch_index(a.tx.order, my);   // records stay indexed by lattice index
                            begin(a.tx, a.ray_begin + rid);
                        }
                    } else {
                        // one transmitter at a time (seldom more than one in a
                        // wavefront), its descriptor read through the scalar cache
                        // (64 rooftop transmitters of up to 1e7 rays: 5.24 -> 5.11 ms
                        // against a search and reads per lane; with refraction
                        // 2 to 4 %)
                        bool todo = mine;
                        while (const unsigned long long m = ballot(todo)) {
                            const int first = __builtin_ctzll(m);
                            const int64_t g = (int64_t)(((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(my >> 32), first) << 32) |
                                                        (unsigned)__builtin_amdgcn_readlane((int)my, first));
                            const int64_t* const prefix = scalar_pointer(a.prefix);
                            if (g < prefix[txi] || g >= prefix[txi + 1]) txi = uniform(find_tx(prefix, a.n_tx, g));
                            const int64_t lo = prefix[txi], hi = prefix[txi + 1];
                            const TxDesc& td = *scalar_pointer(a.txs + txi);
                            if (todo && my >= lo && my < hi) {
                                todo = false;
                                const int64_t n = launch_index(td.order, my - lo);
                                // the geometry tape stays in launch order (a
                                // wavefront of the field pass then reads
                                // consecutive records of nearby directions)
                                rid = MODE == MODE_GEOM ? my : lo + n;
                                tslot = *scalar_pointer(a.slots + txi);
                                mapb = a.map + (int64_t)tslot * a.slot_stride;
                                nlat = n;
                                if (EXT) ikap = 1.0f / td.kappa;
                                begin(td, n);
                            }
                        }
                    }
                }
            }
        }
        if (ballot(active) == 0ull) break;

        // ---- closest hit of the current segment
        int slot = -1, cell = -1;
        float t_hit = INFINITY;
        float w0 = 0.f, w1 = 0.f;
        if (active) {
            const Best best = closest_hit<BRUTE, WIDE, REC>(kernel_args(), o, k, last, stk, lstride, gtid, st_nodes,
                                                            st_tris, st_over);
            slot = best.slot;
            t_hit = best.t;
            if (REC) st_seg++;
            const FwdArgs& a = kernel_args();
            const int W = a.pl.W, H = a.pl.H;
            // ---- plane crossing of this segment
            {
                const float tm = (a.pl.z - o.z) * __builtin_amdgcn_rcpf(k.z);
                const float x = o.x + tm * k.x, y = o.y + tm * k.y;
                const float fx = (x - a.pl.x0) * a.pl.inv_dx, fy = (y - a.pl.y0) * a.pl.inv_dy;
                const bool cross = (k.z != 0.0f) & (tm > 0.0f) & (tm < t_hit) & (fx >= 0.0f) & (fy >= 0.0f) &
                                   (fx < (float)W) & (fy < (float)H);
                cell = cross ? min((int)fy, H - 1) * W + min((int)fx, W - 1) : -1;
                if (REC) st_cross += cross ? 1u : 0u;
                if (FIELDS && cross) {
                    float g = kap * __builtin_amdgcn_rcpf(fabsf(k.z));
                    w0 = g * fs.power(0);
                    if (FIELD == 2 || (FIELD == 0 && a.npol == 2)) w1 = g * fs.power(1);
                }
            }
            if (REC) {
                const int stride = a.L + 1;
                if (a.hits) a.hits[rid * stride + l] = slot >= 0 ? best.id : -1;
                if (a.cells) a.cells[rid * stride + l] = cell;
                if (a.weights) a.weights[rid * stride + l] = w0;
            }
            if (TAPE && a.tape_seg) {
                const int64_t tn = a.tape_n;
                float4* ts = a.tape_seg + (int64_t)l * a.tape_groups * tn + rid;
                ts[0] = make_float4(k.x, k.y, k.z, __int_as_float(slot));
                ts[tn] = make_float4(es.x, es.y, es.z, __int_as_float(cell));
                if constexpr (FIELDS && FIELD == 0) {
                    ts[2 * tn] = make_float4(fs.Ta.re, fs.Ta.im, fs.Tb.re, fs.Tb.im);
                    ts[3 * tn] = make_float4(fs.Tc.re, fs.Tc.im, fs.Td.re, fs.Td.im);
                }
            }
        }

        // ---- deposit (all lanes reconverged here)
        if (FIELDS) {
            const FwdArgs& a = kernel_args();
            const bool two = FIELD == 2 || (FIELD == 0 && a.npol == 2);
            float* const map = MODE == MODE_SINGLE ? a.map : mapb;
            if (a.deposit == 2) {
                // at most kDepositGroups same-cell groups are summed across the
                // wavefront; lanes left over add their own crossings (crossings
                // scattered over many cells would otherwise cost one wavefront
                // reduction per cell)
                unsigned long long pend = ballot(cell >= 0);
                bool done = cell < 0;
                int groups = 0;
                while (pend) {
                    if (groups == kDepositGroups) {
                        if (!done) {
                            unsafeAtomicAdd(map + cell, w0);
                            if (two) unsafeAtomicAdd(map + a.map_stride + cell, w1);
                        }
                        break;
                    }
                    groups++;
                    const int leader = __builtin_ctzll(pend);
                    const int lc = __builtin_amdgcn_readlane(cell, leader);
                    bool mine = !done && cell == lc;
                    // lanes of other transmitters deposit into other maps
                    if (MODE == MODE_MULTI) mine = mine && tslot == __builtin_amdgcn_readlane(tslot, leader);
                    unsigned long long grp = ballot(mine);
                    float v0 = wave_sum(mine ? w0 : 0.0f);
                    float v1 = 0.0f;
                    if (two) v1 = wave_sum(mine ? w1 : 0.0f);
                    // (the address per lane: for a uniform one the compiler would
                    // reduce over the wavefront again)
                    if (lane == leader) {
                        unsafeAtomicAdd(map + cell, v0);
                        if (two) unsafeAtomicAdd(map + a.map_stride + cell, v1);
                    }
                    if (mine) done = true;
                    pend &= ~grp;
                }
            } else if (cell >= 0) {
                unsafeAtomicAdd(map + cell, w0);
                if (two) unsafeAtomicAdd(map + a.map_stride + cell, w1);
            }
        }

        // ---- reflect, or end the ray
        if (active) {
            const FwdArgs& a = kernel_args();
            if (slot < 0 || l == a.L) {
                if (TAPE && a.tape_nseg) a.tape_nseg[rid] = l + 1;
                active = false;
            } else {
                float4 nm = a.normals[slot];
                int mat = __float_as_int(nm.w);
                Bounce b = bounce_geometry(k, es, f3(nm.x, nm.y, nm.z));
                int kind = 0;          // 0 specular reflection, 1 diffuse reflection, 2 transmission
                float3 knew = b.kr, esnew = b.es_new;
                if (FIELDS) {
                    cf eta = cf{a.eps_r[mat], -a.sigma[mat] * a.pl.inv_eps0_omega};
                    Fresnel F = fresnel<false>(b.c, eta);
                    cf cperp = F.rperp, cpar = F.rpar;
                    float qs = 1.0f, s2 = 0.0f;
                    if (EXT) {
                        // single-layer slab: r and t from r' and x = exp(-j q)
                        cf tperp = cf{0.0f, 0.0f}, tpar = cf{0.0f, 0.0f};
                        if (a.thickness) slab(F, a.k0 * a.thickness[mat], tperp, tpar);
                        cperp = F.rperp;
                        cpar = F.rpar;
                        const float Sm = a.scattering ? a.scattering[mat] : 0.0f;
                        if (a.refraction || Sm > 0.0f) {
                            // interaction shares with A = |r|^2, B = |t|^2 (0
                            // without refraction): q(R) = R^2 A/(A+B),
                            // q(S) = S^2 A/(A+B), q(T) = B/(A+B); the sampled
                            // branch carries 1/sqrt(q)
                            const float ar = cabs2(F.rperp) + cabs2(F.rpar);
                            const float at = a.refraction ? cabs2(tperp) + cabs2(tpar) : 0.0f;
                            const float tot = ar + at;
                            const float fa = tot > 0.0f ? ar / tot : 1.0f;
                            s2 = Sm * Sm;
                            const float qr = (1.0f - s2) * fa;
                            qs = s2 * fa;
                            const float u = philox_uniform(a.seed, MODE == MODE_SINGLE ? a.ray_begin + rid : nlat, l, 1u);
                            kind = u < qr ? 0 : (u < qr + qs ? 1 : 2);
                            if (kind != 1) {
                                const float q = kind == 0 ? qr : (tot > 0.0f ? at / tot : 0.0f);
                                // specular share R = sqrt(1 - S^2) (eq. R)
                                const float sc = __builtin_amdgcn_rsqf(q) * (kind == 0 ? sqrtf(1.0f - s2) : 1.0f);
                                cperp = cscale(kind == 2 ? tperp : F.rperp, sc);
                                cpar = cscale(kind == 2 ? tpar : F.rpar, sc);
                                if (kind == 2) knew = k;
                            }
                        }
                    }
                    if (EXT && kind == 1) {
                        if constexpr (EXT && FIELD == 0) {
                            // diffuse reflection (Lambertian): direction drawn over
                            // the hemisphere of the incident side, field scaled by
                            // sqrt(2 cos(theta_s) S^2 Gamma^2 / q(S)) and mixed by
                            // the cross-polarisation matrix with random phases, in
                            // the theta/phi bases of the incident and new direction
                            const cf e0 = cadd(cscale(fs.Ta, fs.c0t), cscale(fs.Tb, fs.c0p));
                            const cf e1 = cadd(cscale(fs.Tc, fs.c0t), cscale(fs.Td, fs.c0p));
                            const cf ap = cadd(cscale(e0, b.w00), cscale(e1, b.w01));
                            const cf al = cadd(cscale(e0, b.w10), cscale(e1, b.w11));
                            const float en2 = cabs2(e0) + cabs2(e1);
                            const float g2 = en2 > 0.0f ? (cabs2(cmul(F.rperp, ap)) + cabs2(cmul(F.rpar, al))) / en2 : 0.0f;
                            const uint4 w = philox4(a.seed, MODE == MODE_SINGLE ? a.ray_begin + rid : nlat, l, 2u);
                            const float cs = word_uniform(w.x), ss = sqrtf(fmaxf(0.0f, 1.0f - cs * cs));
                            float sph, cph, s1, c1, s2p, c2p;
                            sincospif(2.0f * word_uniform(w.y), &sph, &cph);
                            sincospif(2.0f * word_uniform(w.z), &s1, &c1);
                            sincospif(2.0f * word_uniform(w.w), &s2p, &c2p);
                            float3 n = f3(nm.x, nm.y, nm.z);
                            if (dot3(k, n) > 0.0f) n = n * -1.0f;
                            knew = diffuse_direction(n, cs, ss, cph, sph);
                            float3 thi, phi_i, phs;
                            sph_basis(k, thi, phi_i);
                            sph_basis(knew, esnew, phs);
                            const float3 ep = cross3(k, es);
                            const float p00 = dot3(thi, es), p01 = dot3(thi, ep);
                            const float p10 = dot3(phi_i, es), p11 = dot3(phi_i, ep);
                            const float K = a.xpd[mat], sk = sqrtf(K), ck = sqrtf(1.0f - K);
                            const float fw = scatter_weight(a.pattern ? a.pattern + 4 * mat : nullptr, b.c, cs, k, knew, b.kr);
                            const float sc = sqrtf(fw * s2 * g2) * __builtin_amdgcn_rsqf(qs);
                            const float a0 = ck * p00 - sk * p10, a1 = ck * p01 - sk * p11;   // theta row
                            const float b0 = sk * p00 + ck * p10, b1 = sk * p01 + ck * p11;   // phi row
                            const cf x1 = cf{c1 * sc, s1 * sc}, x2 = cf{c2p * sc, s2p * sc};
                            const cf na = cmul(x1, cadd(cscale(fs.Ta, a0), cscale(fs.Tc, a1)));
                            const cf nb = cmul(x1, cadd(cscale(fs.Tb, a0), cscale(fs.Td, a1)));
                            const cf nc = cmul(x2, cadd(cscale(fs.Ta, b0), cscale(fs.Tc, b1)));
                            const cf nd = cmul(x2, cadd(cscale(fs.Tb, b0), cscale(fs.Td, b1)));
                            fs.Ta = na;
                            fs.Tb = nb;
                            fs.Tc = nc;
                            fs.Td = nd;
                        }
                    } else {
                        fs.interact(b, cperp, cpar);
                    }
                }
                o = o + k * t_hit;
                k = knew;
                es = esnew;
                last = slot;
                l++;
                if (EXT) rlen = kind == 1 ? 0.0f : rlen + t_hit;   // a diffuse point starts a new tube
                if constexpr (EXT && FIELD == 0) {
                    if (l >= a.rr_depth && (a.rr_p_max > 0.0f || a.gain_threshold > 0.0f)) {
                        // early termination before segment l: the distance-normalised
                        // gain ||T C||^2 of polarisation 0 (times |alpha|^2)
                        const float gn = fs.power(0) * (kap * (MODE == MODE_SINGLE ? a.inv_kappa : ikap));
                        bool drop = false;
                        if (a.gain_threshold > 0.0f && rlen > 0.0f)
                            drop = a.gain_scale * gn * __builtin_amdgcn_rcpf(rlen * rlen) < a.gain_threshold;
                        if (!drop && a.rr_p_max > 0.0f) {
                            const float p = fminf(gn, a.rr_p_max);
                            if (philox_uniform(a.seed, MODE == MODE_SINGLE ? a.ray_begin + rid : nlat, l, 0u) < p) {
                                const float sc = __builtin_amdgcn_rsqf(p);   // survivors carry 1/sqrt(p)
                                fs.Ta = cscale(fs.Ta, sc);
                                fs.Tb = cscale(fs.Tb, sc);
                                fs.Tc = cscale(fs.Tc, sc);
                                fs.Td = cscale(fs.Td, sc);
                            } else {
                                drop = true;
                            }
                        }
                        if (drop) {
                            active = false;
                            if (TAPE && a.tape_nseg) a.tape_nseg[rid] = l;   // segments 0..l-1 were traced
                        }
                    }
                }
            }
        }
    }

    if (REC) {
        const FwdArgs& a = kernel_args();
        if (a.stats) {
            unsigned long long v[5] = {st_seg, st_cross, st_nodes, st_tris, st_over};
            for (int i = 0; i < 5; i++) {
                unsigned long long s = v[i];
                for (int off = 32; off >= 1; off >>= 1) {
                    unsigned lo = __shfl_xor((unsigned)(s & 0xffffffffu), off);
                    unsigned hi = __shfl_xor((unsigned)(s >> 32), off);
                    s += ((unsigned long long)hi << 32) | lo;
                }
                if (lane == 0 && s) atomicAdd(a.stats + i, s);
            }
        }
    }
}

// Zero the map (unless accumulating), set the heads of the work queues behind
// the wavefronts' first entries and mark the queues that these drain (launched
// with at least two 256-thread blocks, so that the grid has more than RT_QUEUES
// threads).  A kernel, not a memset, so that the whole call can be captured in
// a HIP graph.
__global__ void k_prepare(float* __restrict__ map, int64_t n, unsigned long long* __restrict__ counter, int nq,
                          unsigned long long per_queue, int blocks, int waves_per_block) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    auto head = [&](int q) { return (unsigned long long)((blocks - q + nq - 1) / nq) * (unsigned)waves_per_block; };
    if (i < nq) counter[i * RT_QUEUE_STRIDE] = head((int)i);
    if (i == RT_QUEUES) {
        unsigned long long drained = 0;
        for (int q = 0; q < nq; q++) drained |= head(q) >= per_queue ? 1ull << q : 0ull;
        counter[i * RT_QUEUE_STRIDE] = drained;
    }
    for (; i < n; i += (int64_t)gridDim.x * blockDim.x) map[i] = 0.0f;
}

}  // namespace

// Fewer indices than this are launched in lattice order.
static constexpr int64_t kOrderMin = 512;
// Smallest chunk of the rest: a wavefront of it spans less than half a turn.
static constexpr int kOrderTailMin = 10;      // 144

LaunchOrder rt_launch_order(int64_t count, int64_t N, bool coherent) {
    constexpr FibTable fib = make_fib_table();
    LaunchOrder o{0, 0, 0};
    if (!coherent || count < kOrderMin) return o;
    // wave patches of roughly equal extent in polar and azimuthal angle: a
    // chunk spans 2 F / N in z, a wave 2 pi 64 / F in azimuth -> F^2 ~ 64 pi N
    const double want = std::sqrt(64.0 * RT_PI * (double)N);
    int i = kOrderTailMin;
    while (i + 1 < kFibCount && want * want > (double)fib.e[i].size * (double)fib.e[i + 1].size) i++;
    while (i > kOrderTailMin && (int64_t)fib.e[i].size > count) i--;
    o.chunk = i;
    o.full = count / fib.e[i].size * fib.e[i].size;
    int64_t rest = count - o.full;
    for (int j = i - 1; j >= kOrderTailMin; j--)
        if (rest >= (int64_t)fib.e[j].size) {
            o.tail |= 1u << j;
            rest -= fib.e[j].size;
        }
    return o;
}

int64_t rt_order_chunk(const LaunchOrder& o) {
    constexpr FibTable fib = make_fib_table();
    return o.chunk ? (int64_t)fib.e[o.chunk].size : 1;
}

int rt_persistent_blocks(int block, int device) {
    static int cu[64] = {0};
    int dev = device < 64 ? device : 0;
    if (!cu[dev]) {
        int c = 0;
        if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || c <= 0) c = 256;
        cu[dev] = c;
    }
    // what is resident: four wavefronts per SIMD (registers; 16 of a CU's stacks
    // take 128 KB of LDS)
    int waves_per_cu = 16;
    int blocks_per_cu = std::max(1, waves_per_cu * 64 / block);
    return cu[dev] * blocks_per_cu;
}

static void base_args(FwdArgs& a, const rt_scene* s, int block, const float* eps_r, const float* sigma,
                      const PlaneDesc& pl, int L, float t_min) {
    memset(&a, 0, sizeof(a));
    a.nodes = s->nodes;
    a.wide = s->wide;
    a.n_wide = (int)s->n_wide;
    a.tris = s->tris;
    a.normals = s->normals;
    a.root = s->root;
    a.n_tri = (int)s->n_tri;
    a.eps_r = eps_r;
    a.sigma = sigma;
    a.pl = pl;
    a.L = L;
    a.t_min = t_min;
    a.counter = s->counters;
    a.spill = s->spill;
    a.tape_groups = 4;
    a.npol = 1;
    a.refill = 1;
}

// 4-wide nodes of a tree that fills an L2 of 4 MB.
static constexpr int64_t kLargeTree = 32768;

// Grid, work queues and spill area of one launch of a.n_work rays.
static rt_status size_launch(FwdArgs& a, const rt_scene* s, int block, const LaunchOrder& order, bool brute,
                             int* blocks_out) {
    const int per_block = block / 64;
    int64_t blocks = rt_persistent_blocks(block, s->device);
    int64_t waves = blocks * per_block;
    // fewer rays than the resident wavefronts have lanes: narrower wavefronts
    // (whose lanes wait less for each other), at least 8 rays wide; not where
    // every triangle is tested, for as long on each lane (5,810 triangles, 2e4
    // rays: 11.4 ms with 8 rays per wavefront, 8.6 with 64).
    // Nor on a map of so few cells that every wavefront adds to the same ones (25 ns
    // each on one address), in a scene of so few triangles that this takes longer
    // than its rays (14 triangles, 1 cell, 2e4 rays 46 -> 20 us, 1e5 52 ->
    // 33; city, 1 cell: 2e4 rays would take 108 us instead of 101).
    const bool crowded = a.tape_groups == 4 && a.map_stride <= 256 && s->n_wide < 32;
    a.width = 64;
    while (!brute && !crowded && a.width > 8 && a.n_work <= (waves - 7) * (a.width / 2)) a.width /= 2;
    a.n_units = (a.n_work + a.width - 1) / a.width;
    // one transmitter on a large tree, with room for narrow first units on both
    // sides of the equator
    const int64_t equator = a.n_tx == 1 ? a.n_work / 2 : a.tx.n_rays / 2 - a.ray_begin;
    const bool narrow_first = a.n_tx <= 1 && s->n_wide >= kLargeTree && equator > 8 * waves + 256 &&
                              a.n_work - equator > 8 * waves + 256;
    a.once = (a.n_units + 7) / 8 * 8 <= waves && !(narrow_first && a.width > 16);
    a.mid = -1;
    a.nq = 1;
    a.run = 1;
    a.claim = a.width;
    a.first_width = a.width;
    unsigned n_stretch = 0;        // stretches per queue that come in turn, 0 = one front
    int64_t stretch = 0;           // units in each
    if (a.once) {
        blocks = std::max<int64_t>(1, ((a.n_units + 7) / 8 * 8 + per_block - 1) / per_block);
    } else {
        // claims on one head follow each other at 25 ns, 16 heads keep up with the
        // shortest rays (14 triangles, 3e6 rays: 124 us with 8, 101 us with 16);
        // more heads cost the wavefronts more looks at the end
        a.nq = 16;
        if (const char* env = getenv("RTMAP_QUEUES"))
            a.nq = std::max(1, std::min(RT_QUEUES, atoi(env)));
        a.nq = (int)std::min<int64_t>(a.nq, blocks);
        // units small enough that every wavefront runs about 16 of them, large
        // enough to keep queue atomics rare; whole multiples of the wavefront,
        // so that a refill stays on one stretch of the launch order
        a.claim = 64 * (int)std::max<int64_t>(1, std::min<int64_t>(4, a.n_units / (waves * 16)));
        if (const char* env = getenv("RTMAP_CLAIM"))
            a.claim = std::max(64, std::min(4096, atoi(env)));
        // units, and so entries, are numbered in 32 bits
        while (a.n_work / a.claim >= (int64_t)1 << 30) a.claim *= 2;
        // stretches in turn (see queue_entry) where deposits would meet, but for a
        // geometry tape, which takes none
        if (a.tape_groups == 4 && a.n_units >= 4 * waves) {
            if (a.deposit == RT_DEPOSIT_ATOMIC) n_stretch = 16;
            else if (order.chunk == 0) n_stretch = a.n_tx > 0 ? 8 : 1;
            // a map of a few cells (5,810 triangles, 1 cell, 4e6 rays 853 -> 773 us, 1e7
            // 1.98 -> 1.76 ms; from 64 cells on, and on the 1.02 M-triangle scene, one
            // front is as fast or faster)
            else if (a.map_stride < 32 && s->n_wide < kLargeTree) n_stretch = 4;
        }
        // and where the transmitters' horizons would follow one another
        if (!n_stretch && a.n_tx > 1 && s->n_wide >= kLargeTree && a.n_units <= waves * std::min(64, 8 * a.n_tx)) {
            if (a.n_units >= 4 * waves) n_stretch = 4;
            else if (a.n_tx >= 4) n_stretch = 1;
        }
        const int64_t turn = (int64_t)a.nq * std::max(1u, n_stretch);
        const int64_t narrow = a.n_tx > 1 && !n_stretch ? 32 * waves * a.width : 0;     // indices left to units of one wavefront
        if (a.n_tx > 1) {
            a.n_units = std::max<int64_t>(0, a.n_work - narrow) / a.claim / turn * turn;
        } else {
            a.n_units = (a.n_work + a.claim - 1) / a.claim;
            a.mid = std::min(a.n_units, std::max<int64_t>(0, equator / a.claim));
            // narrow first units, a whole number of the others on both sides of mid
            const int64_t hole = 16 * waves, side = hole / 2 / a.claim;
            if (narrow_first && a.n_units <= 6 * waves * 64 / a.claim && blocks % a.nq == 0 &&
                hole % (2 * a.claim) == 0 && a.mid >= side && a.n_units - a.mid > side) {
                a.first_width = 16;
                a.n_first = (unsigned)(waves / a.nq);
                a.mid -= side;
                a.n_units -= 2 * side;
                a.hole = a.mid * a.claim;
                a.hole_size = hole;
            }
            a.run = (unsigned)std::max<int64_t>(1, rt_order_chunk(order) / (2 * a.claim * a.nq));
        }
        stretch = (a.n_units + turn - 1) / turn;
    }
    if (n_stretch) {
        a.run = n_stretch;
        a.n_claim = a.n_run = (unsigned)(n_stretch * stretch);
        a.by_r = 1;
        a.by_k = (unsigned)(a.nq * stretch);
        a.by_q = (unsigned)stretch;
    } else {
        a.n_claim = (unsigned)((a.n_units + a.nq - 1) / a.nq);
        // whole turns of every queue, so that the rest is a stretch of its own
        a.n_run = (unsigned)(a.n_units / ((int64_t)a.run * a.nq)) * a.run;
        a.by_r = (unsigned)a.nq * a.run;
        a.by_k = 1;
        a.by_q = a.run;
    }
    const int64_t rest = std::max<int64_t>(0, a.n_work - a.hole_size - (int64_t)a.n_claim * a.nq * a.claim);
    a.per_queue = (unsigned long long)a.n_first + a.n_claim + (unsigned long long)((rest + (int64_t)a.width * a.nq - 1) / ((int64_t)a.width * a.nq));
    const int64_t threads = blocks * block;
    int64_t need_depth = std::max<int64_t>(0, rt_stack_need(s) - RT_STACK_LDS);
    if ((int64_t)s->spill_entries < need_depth * threads)
        return rt_fail(RT_EOVERFLOW, "traversal spill area too small for this launch");
    a.spill_stride = threads;
    a.spill_depth = (int)need_depth;
    *blocks_out = (int)blocks;
    return RT_OK;
}

template <int MODE>
static void launch_mode(const FwdArgs& a, int accel, bool wide, int blocks, int block, hipStream_t st,
                        bool ext = false) {
    const size_t lds = sizeof(int2) * RT_STACK_LDS * block;   // {node, entry distance} per entry
    // calls with records, statistics or a tape, and the extensions, carry the
    // transfer matrix; the others the fields themselves
    [[maybe_unused]] const bool rec = a.hits || a.cells || a.weights || a.stats || (MODE == MODE_SINGLE && a.tape_seg);
    [[maybe_unused]] const bool two = a.npol == 2;
#define RT_LAUNCH(BRUTE, WIDE, EXT, REC, FIELD) \
    hipLaunchKernelGGL((k_forward<BRUTE, MODE, WIDE, EXT, REC, FIELD>), dim3(blocks), dim3(block), lds, st, a)
    if constexpr (MODE == MODE_GEOM) {
        if (wide) RT_LAUNCH(false, true, false, false, 1);
        else RT_LAUNCH(false, false, false, false, 1);
    } else if constexpr (MODE == MODE_MULTI) {
        if (ext && wide) RT_LAUNCH(false, true, true, false, 0);
        else if (ext) RT_LAUNCH(false, false, true, false, 0);
        else if (wide) RT_LAUNCH(false, true, false, false, 1);
        else RT_LAUNCH(false, false, false, false, 1);
    } else if (accel == RT_ACCEL_BRUTE) {
        if (ext) RT_LAUNCH(true, false, true, true, 0);
        else RT_LAUNCH(true, false, false, true, 0);
    } else if (!wide) {
        if (ext) RT_LAUNCH(false, false, true, true, 0);
        else RT_LAUNCH(false, false, false, true, 0);
    } else if (ext) {
        if (rec) RT_LAUNCH(false, true, true, true, 0);
        else RT_LAUNCH(false, true, true, false, 0);
    } else if (rec) {
        RT_LAUNCH(false, true, false, true, 0);
    } else if (two) {
        RT_LAUNCH(false, true, false, false, 2);
    } else {
        RT_LAUNCH(false, true, false, false, 1);
    }
#undef RT_LAUNCH
}

// Tree width: forced by accel, else tuned (or overridden), default 4-wide.
static bool use_wide(const rt_scene* s, int accel = RT_ACCEL_BVH) {
    if (!s->wide || s->root < 0 || accel == RT_ACCEL_BVH2 || accel == RT_ACCEL_BRUTE) return false;
    if (accel == RT_ACCEL_BVH4) return true;
    if (const char* env = getenv("RTMAP_WIDTH")) return atoi(env) != 2;
    return s->tuned_width != 2;
}

rt_status rt_launch_forward(const FwdLaunch& f, hipStream_t st) {
    const rt_scene* s = f.scene;
    FwdArgs a;
    base_args(a, s, f.block, f.eps_r, f.sigma, f.pl, f.L, f.t_min);
    a.tx = f.tx;
    a.ray_begin = f.ray_begin;
    a.n_work = f.ray_end - f.ray_begin;
    a.deposit = f.deposit;
    a.npol = f.tx.pol == RT_POL_DUAL ? 2 : 1;
    a.map = f.map;
    a.map_stride = (int64_t)f.pl.W * f.pl.H;
    a.tape_seg = f.tape ? f.tape->seg : nullptr;
    a.tape_nseg = f.tape ? f.tape->nseg : nullptr;
    a.tape_n = f.tape ? f.tape->n_rays : 0;
    a.hits = f.hits;
    a.cells = f.cells;
    a.weights = f.weights;
    a.stats = f.stats;
    a.refill = std::max(1, std::min(64, f.refill));
    int blocks = 0;
    rt_status r = size_launch(a, s, f.block, f.tx.order, f.accel == RT_ACCEL_BRUTE, &blocks);
    if (r != RT_OK) return r;
    int64_t map_n = a.map_stride * a.npol;
    {
        int64_t zn = f.zero_map ? map_n : 0;
        int g = (int)std::min<int64_t>(2048, std::max<int64_t>(2, (zn + 255) / 256));
        hipLaunchKernelGGL(k_prepare, dim3(g), dim3(256), 0, st, f.map, zn, s->counters, a.nq,
                           a.per_queue, blocks, f.block / 64);
    }
    a.rr_depth = f.rr_depth;
    a.rr_p_max = f.rr_p_max;
    a.gain_threshold = f.gain_threshold;
    a.seed = f.seed;
    a.gain_scale = f.gain_scale;
    a.inv_kappa = 1.0f / f.tx.kappa;
    a.thickness = f.thickness;
    a.scattering = f.scattering;
    a.xpd = f.xpd;
    a.pattern = f.pattern;
    a.refraction = f.refraction;
    a.k0 = f.k0;
    const bool ext = f.rr_p_max > 0.0f || f.gain_threshold > 0.0f || f.thickness != nullptr || f.scattering != nullptr;
    if (a.n_work > 0) launch_mode<MODE_SINGLE>(a, f.accel, use_wide(s, f.accel), blocks, f.block, st, ext);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return rt_hip_fail(e, "forward launch");
    return RT_OK;
}

// Several transmitters in one persistent launch.  geom_only = false: deposit
// into maps[slot] (one material set, map stride slot_stride, maps zeroed
// here); geom_only = true: write the geometry tape (2 records per segment).
rt_status rt_launch_forward_multi(const rt_scene* s, const float* eps_r, const float* sigma, const PlaneDesc& pl,
                                  int L, float t_min, int block, int deposit, int refill,
                                  const TxDesc* txs, const int64_t* prefix, const int32_t* slots, int n_tx,
                                  const LaunchOrder& order, int64_t total_rays, bool geom_only, float* maps, int64_t slot_stride, int64_t zero_floats,
                                  float4* geom_seg, int* geom_nseg, const FwdExt* ext, hipStream_t st) {
    FwdArgs a;
    base_args(a, s, block, eps_r, sigma, pl, L, t_min);
    a.ray_begin = 0;
    a.n_work = total_rays;
    a.deposit = deposit;
    a.map = maps;
    a.map_stride = (int64_t)pl.W * pl.H;
    a.txs = txs;
    a.prefix = prefix;
    a.slots = slots;
    a.n_tx = n_tx;
    a.slot_stride = slot_stride;
    a.refill = std::max(1, std::min(64, refill));
    if (geom_only) {
        a.tape_seg = geom_seg;
        a.tape_nseg = geom_nseg;
        a.tape_n = total_rays;
        a.tape_groups = 2;
    }
    int blocks = 0;
    rt_status r = size_launch(a, s, block, order, false, &blocks);
    if (r != RT_OK) return r;
    int g = (int)std::min<int64_t>(4096, std::max<int64_t>(2, (zero_floats + 255) / 256));
    hipLaunchKernelGGL(k_prepare, dim3(g), dim3(256), 0, st, maps, zero_floats, s->counters, a.nq,
                       a.per_queue, blocks, block / 64);
    bool use_ext = false;
    if (ext && !geom_only) {
        a.rr_depth = ext->rr_depth;
        a.rr_p_max = ext->rr_p_max;
        a.gain_threshold = ext->gain_threshold;
        a.gain_scale = ext->gain_scale;
        a.seed = ext->seed;
        a.thickness = ext->thickness;
        a.scattering = ext->scattering;
        a.xpd = ext->xpd;
        a.pattern = ext->pattern;
        a.refraction = ext->refraction;
        a.k0 = ext->k0;
        use_ext = ext->rr_p_max > 0.0f || ext->gain_threshold > 0.0f || ext->thickness != nullptr ||
                  ext->scattering != nullptr;
    }
    if (total_rays > 0) {
        if (geom_only) launch_mode<MODE_GEOM>(a, RT_ACCEL_BVH, use_wide(s), blocks, block, st);
        else launch_mode<MODE_MULTI>(a, RT_ACCEL_BVH, use_wide(s), blocks, block, st, use_ext);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return rt_hip_fail(e, "batched forward launch");
    return RT_OK;
}
