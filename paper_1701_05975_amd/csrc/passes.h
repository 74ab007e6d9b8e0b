// passes.h -- the per-source steps of weighted Brandes, written as wave-level
// routines over a list of vertices.  The batched form calls them with the
// waves of one workgroup and counters in LDS; the plain form with every wave
// of the grid and counters in global memory.
//
// Mapping of work to lanes (the warp-centric idea of Sec. 3.4 recast for
// 64-lane wavefronts): the expansion lays the arcs of up to 64 queued vertices
// out flat over the wave, so that every lane has an arc whatever the degrees
// are, and a hub's arcs over the whole workgroup; the batched form's count and
// dependency passes do the same where a vertex has more than one arc to look
// at (the plain form's use a lane, a group of lanes or the wave per vertex).
// Only queued vertices get lanes (the work-efficient queue of
// Sec. 3.3); a fixed group width and a scan over every vertex (node-parallel)
// are selectable for comparison.
#pragma once

#include "dev_common.h"

template <int SCOPE>
__device__ __forceinline__ uint32_t atomic_min_u32(uint32_t *p, uint32_t v)
{
    return __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, SCOPE);
}

template <int SCOPE>
__device__ __forceinline__ uint32_t dist_min(const Slab &S, uint32_t u, uint32_t v)
{
    if ((int32_t)u < S.H) {
        if (S.w8) {
            // 8-bit entry (see LDS8_WIN): compare-and-swap its word.  v lies
            // above the base (it is offered from the band being expanded), so
            // an entry of 0 (settled below the base) is already smaller.
            // Entries only move down (unreached, then kept in d[] or a value
            // in the window, then smaller values), so the loop ends.
            lds_u32 *wp = lds_ptr(S.ld) + (u >> 2);
            const uint32_t sh = (u & 3u) * 8u;
            const uint32_t fit = v - S.base8 + 1u; // window code of v, if at most LDS8_WIN
            uint32_t cur = *wp;
            for (;;) {
                const uint32_t h = (cur >> sh) & 0xffu;
                if (h - 1u < LDS8_WIN && S.base8 + h - 1u <= v)
                    return S.base8 + h - 1u; // already at most v
                if (h == 0u)
                    return 0u;
                if (fit > LDS8_WIN && h == LDS8_FAR) // kept in d[]
                    return atomic_min_u32<SCOPE>(&S.d[u], v);
                // h is unreached, kept in d[] while v fits, or a larger value
                const uint32_t e = fit <= LDS8_WIN ? fit : LDS8_FAR;
                const uint32_t nw = (cur & ~(0xffu << sh)) | (e << sh);
                uint32_t expect = cur;
                if (__hip_atomic_compare_exchange_strong(wp, &expect, nw, __ATOMIC_RELAXED,
                                                         __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_WORKGROUP)) {
                    // first value that does not fit (h was unreached), or first that
                    // does (h was kept in d[]): d[u] orders these two, so that
                    // exactly one offer sees each earlier value as the old one
                    if (e == LDS8_FAR || h == LDS8_FAR)
                        return atomic_min_u32<SCOPE>(&S.d[u], v);
                    return h - 1u < LDS8_WIN ? S.base8 + h - 1u : BC_INF;
                }
                cur = expect;
            }
        }
        if (!S.w16)
            return __hip_atomic_fetch_min(lds_ptr(S.ld) + u, v, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_WORKGROUP);
        // 16-bit entry: LDS has no 16-bit minimum, so compare-and-swap the
        // 32-bit word holding it.  Entries only move down (unreached, then
        // kept in d[], then a value below LDS16_FAR, then smaller values), and
        // each failed swap saw another lane move one of the word's two
        // entries, so the loop ends.
        lds_u32 *wp = lds_ptr(S.ld) + (u >> 1);
        const uint32_t sh = (u & 1u) * 16u;
        uint32_t cur = *wp;
        for (;;) {
            const uint32_t h = (cur >> sh) & 0xffffu;
            if (h < LDS16_FAR && h <= v)
                return h; // already at most v
            if (v >= LDS16_FAR && h == LDS16_FAR) // kept in d[]
                return atomic_min_u32<SCOPE>(&S.d[u], v);
            // h is unreached, or kept in d[] while v fits, or a larger value
            const uint32_t e = v < LDS16_FAR ? v : LDS16_FAR;
            const uint32_t nw = (cur & ~(0xffffu << sh)) | (e << sh);
            uint32_t expect = cur;
            if (__hip_atomic_compare_exchange_strong(wp, &expect, nw, __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_WORKGROUP)) {
                // as for the 8-bit entries: d[u] orders the offers around LDS16_FAR
                if (e == LDS16_FAR || h == LDS16_FAR)
                    return atomic_min_u32<SCOPE>(&S.d[u], v);
                return h < LDS16_FAR ? h : BC_INF;
            }
            cur = expect;
        }
    }
    return atomic_min_u32<SCOPE>(&S.d[u], v);
}

template <int SCOPE>
__device__ __forceinline__ int atomic_xchg_i32(int32_t *p, int32_t v)
{
    return __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, SCOPE);
}

template <int SCOPE>
__device__ __forceinline__ int atomic_or_i32(int32_t *p, int32_t v)
{
    return __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, SCOPE);
}

template <int SCOPE>
__device__ __forceinline__ uint64_t load_u64(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, SCOPE);
}

template <int SCOPE>
__device__ __forceinline__ void store_u64(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, SCOPE);
}

template <int SCOPE>
__device__ __forceinline__ double load_f64(const double *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, SCOPE);
}

template <int SCOPE>
__device__ __forceinline__ void store_f64(double *p, double v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, SCOPE);
}

// ---------------------------------------------------------------------------
// Forward pass, frontier expansion (Alg. 2 relaxation step over the queue of
// Alg. 5; near-far banding instead of the Eq. 4 settle rule).
//
// Every arc (v, u, w) of a queued vertex v proposes d[v] + w for u; atomicMin
// keeps the least.  A lane that lowered d[u] below the band threshold puts u
// in the next near queue (once per queue, by tag) and, the first time, in the
// band's member list; a lower value at or above the threshold sends u to the
// far pile (once): the inner pile below the pile bound, else the outer pile,
// which is only scanned when the threshold passes the bound.  What is the
// first time follows from the value that the minimum replaced.
// ---------------------------------------------------------------------------
// Steps of 64 arcs whose loads are in flight together: with a lane's load
// behind a branch the compiler waits for it there, and the steps' latencies
// added up.  1024 sources of R-MAT scale 20: 262 ms at one step, 235 at two, 225
// at four, 223 at six; a Kronecker graph of scale 16 (1024 threads) 6.4 / 6.5
// / 6.9 ms at two, four and six, the grid 87 / 88 / 88.
#ifndef EXPAND_UNROLL
#define EXPAND_UNROLL 4
#endif

struct ExpandCtx {
    const int32_t *items;
    int len;
    int all_vertices;     // node-parallel: scan every vertex, expand those queued now
    int32_t cur_tag;      // tag of the queue being expanded (node-parallel filter)
    int vw;               // 0: arcs laid out flat; else a fixed group of vw lanes per vertex
    int worker, nworkers; // wave index and wave count over the item list
    uint32_t *marks;      // 2 EXPAND_UNROLL words of LDS of this wave (flat_starts)
    uint32_t thr;         // band threshold: d < thr is near
    int32_t tag_next;     // tag of the queue being filled
    int32_t *next_q;
    int *next_cnt;
    int32_t *order;
    int *order_cnt;
    int32_t *far_q;
    int *far_cnt;
    uint32_t bound;       // far values at or above go to the outer pile (BC_INF: none)
    int32_t *outer_q;
    int *outer_cnt;
    int32_t *huge_q;      // optional: vertices with more than wg_deg arcs are listed here
    int *huge_cnt;        // for the whole workgroup or team to expand after the pass
    int keys;             // record each vertex's (distance, predecessor) key and ties
    const uint32_t *trow; // with keys: in-row offsets, whose slices hold the tie entries
    uint32_t wg_deg;
    // Far-bucket ring (batched form, relax<.., true>; else the two-tier pile above).  A far
    // value below `bound` goes to bucket value / bdelta, slot bucket % nbk,
    // when the value it replaces lay in a higher bucket (or beyond the ring);
    // a full bucket sends the vertex to the outer pile and sets *forced, so
    // that the pile is scanned at the next band change.
    int32_t *bk;
    int *bcnt;
    uint32_t bdelta;
    int nbk, bcap;
    int *forced;
};

// Predecessor keys (batched form).  While distances are being found, the
// dependency field of a vertex (unused until its count is taken) holds the
// least (distance << 32 | tail) over the improvements it received, and the
// bits from TIE_SHIFT up in its flags word count the relaxations that
// matched its distance at the time (ties).  A relaxation that offers v its
// final distance comes from a tight arc whose tail is at its own final
// distance (one from a larger tail distance offers more), and it always
// leaves an event: exactly one of them lowers d[v] to that value, and is the
// key, each other one is a tie.  Ties at a larger distance belong to values
// that were improved on later.  So the key's tail and the tails of the ties
// at the key's distance name every shortest-path predecessor, each once per
// tight arc and per expansion of its tail at that distance: a tail improved
// while it is being expanded can be expanded again at the same distance.
//
// The first TIE_MAX ties of a vertex are kept as (distance, tail) pairs in
// its own slice of preds[] (two words each, as far as the slice holds them),
// which the count pass reads until it writes the vertex's DAG list there.  A
// vertex whose ties were all kept and whose predecessor tails are all
// distinct takes its count and its DAG list from the key and those pairs
// without reading its in-arcs.  A vertex with
// more ties, or with a tail seen twice (a second expansion, or parallel tight
// arcs: the pairs cannot tell these apart), scans its in-arcs.
#define VFLAG_OUTER 2 // in the outer far pile (bucket ring only)
#define VFLAG_LIST 4  // the DAG list (or the only predecessor) of v is recorded
#define TIE_SHIFT 4
#define TIE_MAX 7
#define KEY_NONE (~0ull)

__device__ __forceinline__ uint64_t *key_ptr(const Slab &S, int32_t v)
{
    return reinterpret_cast<uint64_t *>(&S.delta[v]);
}

// Arcs handled per step by a lane that walks its own row: their heads and
// the heads' distances are loaded together, so several independent loads per
// lane are in flight instead of one dependent chain per arc.
#ifndef LANE_UNROLL
#define LANE_UNROLL 2
#endif

// Lanes of a group that counts one vertex of medium in-degree.
#ifndef EXPAND_GROUP
#define EXPAND_GROUP 16
#endif
// Hubs (batched form): a vertex with more than wg_deg arcs (default
// BC_HUB_DEG) is expanded by every wave of the workgroup after the pass, so
// that it does not keep one wave busy while the others wait at the barrier.
// The list holds EXPAND_WG_CAP vertices (a team's, in global memory,
// EXPAND_TEAM_CAP); further ones stay with their wave.
#define EXPAND_WG_CAP 256
#define EXPAND_TEAM_CAP 4096

template <int SCOPE> constexpr int hub_cap()
{
    return SCOPE == __HIP_MEMORY_SCOPE_AGENT ? EXPAND_TEAM_CAP : EXPAND_WG_CAP;
}

// Offers nd to u from tail (lanes with `cand`); called by whole waves.
template <int SCOPE, bool BKT = false>
__device__ __forceinline__ void relax_commit(const Slab &S, const ExpandCtx &c, bool cand,
                                             uint32_t u, uint32_t nd, uint32_t tail,
                                             uint32_t &far_min, uint32_t &outer_min,
                                             uint64_t &nimp)
{
    bool imp = false, tie = false;
    uint32_t was = BC_INF;
    if (cand) {
        was = dist_min<SCOPE>(S, u, nd);
        imp = nd < was;
        tie = nd == was;
    }
    if (c.keys) {
        if (imp) {
            // A resident vertex's improvements follow one another in LDS, so its
            // last store is nearly always that of the least distance: the count
            // pass compares the two and scans the in-arcs if it is not.  The
            // others' check would cost a random read per visit: with plain
            // stores for them too the 1000 x 1000 grid takes 108 ms, not 87, and
            // R-MAT scale 20 226 ms, not 213.
            const uint64_t key = (uint64_t)nd << 32 | tail;
            if ((int32_t)u < S.H)
                __hip_atomic_store(key_ptr(S, (int32_t)u), key, __ATOMIC_RELAXED, SCOPE);
            else
                __hip_atomic_fetch_min(key_ptr(S, (int32_t)u), key, __ATOMIC_RELAXED, SCOPE);
        }
        // counting stops past TIE_MAX (beyond it a vertex scans anyway), so
        // the count stays below TIE_MAX + 2 + the threads of the workgroup
        if (tie && ((uint32_t)__hip_atomic_load(&S.flags[u], __ATOMIC_RELAXED, SCOPE) >>
                    TIE_SHIFT) <= TIE_MAX) {
            const uint32_t t = (uint32_t)__hip_atomic_fetch_add(&S.flags[u], 1 << TIE_SHIFT,
                                                                __ATOMIC_RELAXED, SCOPE) >>
                               TIE_SHIFT;
            if (t < TIE_MAX) {
                const uint32_t tb = c.trow[u], te = c.trow[u + 1];
                if (tb + 2 * (t + 1) <= te) {
                    S.preds[tb + 2 * t] = (int32_t)nd;
                    S.preds[tb + 2 * t + 1] = (int32_t)tail;
                }
            }
        }
    }
    // The old value says where u stands already: offers to one vertex take
    // effect one after another, so exactly one of them sees each step down.
    bool pn = false, pm = false, pf = false, po = false;
    int bslot = -1; // far-bucket ring: the slot u goes to
    if (imp) {
        ++nimp;
        const uint32_t old = was;
        if (nd < c.thr) {
            pn = (int32_t)u < S.HQ
                     ? qbit_set(S, u)
                     : atomic_xchg_i32<SCOPE>(&S.stamp[u], c.tag_next) != c.tag_next;
            pm = old >= c.thr; // first value below the band threshold
        } else if (nd < c.bound) {
            if (BKT) {
                const uint32_t b = nd / c.bdelta;
                if (old == BC_INF || old >= (b + 1u) * c.bdelta)
                    bslot = (int)(b % (uint32_t)c.nbk);
            } else {
                far_min = nd < far_min ? nd : far_min;
                pf = old >= c.bound;
            }
        } else {
            outer_min = nd < outer_min ? nd : outer_min;
            po = old == BC_INF;
            if (BKT && po)
                po = (atomic_or_i32<SCOPE>(&S.flags[u], VFLAG_OUTER) & VFLAG_OUTER) == 0;
        }
    }
    if (BKT && __ballot(bslot >= 0)) {
        if (bslot >= 0) {
            const int k = atomicAdd(&c.bcnt[bslot], 1);
            if (k < c.bcap) {
                c.bk[(size_t)bslot * (size_t)c.bcap + (size_t)k] = (int32_t)u;
            } else { // a full bucket: the outer pile keeps u until the next band change
                *c.forced = 1;
                outer_min = nd < outer_min ? nd : outer_min;
                po = (atomic_or_i32<SCOPE>(&S.flags[u], VFLAG_OUTER) & VFLAG_OUTER) == 0;
            }
        }
    }
    if (__ballot(imp)) {
        // one atomic instruction for all four counters: lane i adds the i-th
        const uint64_t mn = __ballot(pn), mm = __ballot(pm), mf = __ballot(pf), mo = __ballot(po);
        const int lane = lane_id();
        int *const c0 = c.next_cnt, *const c1 = c.order_cnt, *const c2 = c.far_cnt,
                   *const c3 = c.outer_cnt;
        int *const at = lane == 0 ? c0 : lane == 1 ? c1 : lane == 2 ? c2 : c3;
        const int add = __popcll(lane == 0 ? mn : lane == 1 ? mm : lane == 2 ? mf : mo);
        int base = 0;
        if (lane < 4 && add > 0)
            base = atomicAdd(at, add);
        const int b0 = __builtin_amdgcn_readlane(base, 0), b1 = __builtin_amdgcn_readlane(base, 1),
                  b2 = __builtin_amdgcn_readlane(base, 2), b3 = __builtin_amdgcn_readlane(base, 3);
        if (pn)
            c.next_q[b0 + (int)lanes_below(mn)] = (int32_t)u;
        if (pm)
            c.order[b1 + (int)lanes_below(mm)] = (int32_t)u;
        if (pf)
            c.far_q[b2 + (int)lanes_below(mf)] = (int32_t)u;
        if (po)
            c.outer_q[b3 + (int)lanes_below(mo)] = (int32_t)u;
    }
}

// Fixed virtual-warp mapping (Sec. 3.4): a group of vw lanes per vertex,
// striding over its arcs; vw = 1 is one thread per vertex, vw = 64 one wave.
template <bool PACKED, int SCOPE, bool BKT = false>
__device__ __forceinline__ void expand_pass_vw(const DevGraph &g, const Slab &S, const ExpandCtx &c,
                               int W, uint32_t &far_min, uint32_t &outer_min, uint64_t &nimp)
{
    const int groups = WAVE / W;
    const int lane = lane_id(), grp = lane / W, sub = lane % W;
    const int len = c.all_vertices ? g.n : c.len;
    for (int base = c.worker * groups; base < len; base += c.nworkers * groups) {
        const int i = base + grp;
        bool valid = i < len;
        int v = 0;
        if (valid) {
            v = c.all_vertices ? i : c.items[i];
            if (c.all_vertices)
                valid = S.stamp[v] == c.cur_tag;
        }
        uint32_t beg = 0, end = 0, dv = BC_INF;
        if (valid) {
            beg = g.row[v];
            end = g.row[v + 1];
            if (v < S.HQ && sub == 0)
                qbit_clear(S, (uint32_t)v);
            // no lane of the group reads the distance before its first lane has cleared
            // the bit: an improvement between the two would leave that lane with the old
            // value (a fence of the wave costs nothing; a wave barrier behind this branch
            // cost small grids 1.4%)
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            dv = dist_get(S, v);
        }
        for (uint32_t e = beg + sub; __ballot(e < end); e += W) { // the whole wave together
            uint32_t u = 0, w = 0;
            bool ok = e < end;
            if (ok) {
                arc_at<PACKED>(g.arc, g.wt, e, g.wshift, g.wmask, u, w);
                ok = dv + w <= dist_peek(S, u);
            }
            relax_commit<SCOPE, BKT>(S, c, ok, u, dv + w, (uint32_t)v, far_min, outer_min, nimp);
        }
    }
}

// Candidates of one wave: offers that the pre-check found no worse than the
// head's distance, held in registers, lane i holding the i-th, until 64 of
// them can be committed together.  Only one arc in ten (Barabasi-Albert,
// n = 100,000) to thirteen (R-MAT scale 20) improves its head, but nearly
// every step of 64 arcs holds one, and a commit is a chain of an LDS or
// global atomic, a returning tag atomic and queue appends: committing each
// step's few cost that chain for every step.  Collected, a wave commits once
// per 64 candidates.  With the flat arcs (the tiers by degree left half of
// the lanes without an arc on those graphs): Barabasi-Albert, 4096 sources,
// 196 -> 169 ms; R-MAT scale 20, 1024 sources, 400 -> 326 ms; Kronecker scale
// 16, 256 sources, 27.4 -> 18.9 ms.
struct CandBuf {
    uint32_t u, nd, tail;
    int cnt; // uniform
};

// Adds the lanes' candidates (called by the whole wave).  The permutation
// sends candidates to the next free lanes and the other lanes to the rest.
template <int SCOPE, bool BKT>
__device__ __forceinline__ void cand_add(const Slab &S, const ExpandCtx &c, CandBuf &b, bool cand,
                                         uint32_t u, uint32_t nd, uint32_t tail, uint32_t &far_min,
                                         uint32_t &outer_min, uint64_t &nimp)
{
    const uint64_t mask = __ballot(cand);
    if (mask == 0)
        return;
    const int lane = lane_id();
    const int p = __popcll(mask);
    const int below = (int)lanes_below(mask);
    const int dst = ((b.cnt + (cand ? below : p + lane - below)) & (WAVE - 1)) << 2;
    const uint32_t ru = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)u);
    const uint32_t rnd = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)nd);
    const uint32_t rt = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)tail);
    const bool fresh = ((lane - b.cnt) & (WAVE - 1)) < p; // received a candidate
    if (b.cnt + p < WAVE) {
        if (fresh) {
            b.u = ru;
            b.nd = rnd;
            b.tail = rt;
        }
        b.cnt += p;
        return;
    }
    const bool low = lane < b.cnt;
    relax_commit<SCOPE, BKT>(S, c, true, low ? b.u : ru, low ? b.nd : rnd, low ? b.tail : rt,
                             far_min, outer_min, nimp);
    b.cnt += p - WAVE;
    b.u = ru;
    b.nd = rnd;
    b.tail = rt;
}

template <int SCOPE, bool BKT>
__device__ __forceinline__ void cand_flush(const Slab &S, const ExpandCtx &c, CandBuf &b,
                                           uint32_t &far_min, uint32_t &outer_min, uint64_t &nimp)
{
    if (b.cnt > 0)
        relax_commit<SCOPE, BKT>(S, c, lane_id() < b.cnt, b.u, b.nd, b.tail, far_min, outer_min,
                                 nimp);
    b.cnt = 0;
}

// Flat layout: items 0 .. items-1 (one per lane, the first lanes) hold the
// flat positions from the strictly increasing offsets `off` on.  starts[j] gets
// the positions in [q0 + 64 j, q0 + 64 j + 64) where an item starts (uniform),
// the result is the number of items that start before q0.  `marks` is 2 N
// words of LDS of this wave (an OR over the lanes by DPP takes about 30
// instructions per 64 positions, which showed in the expansion).
template <int N>
__device__ __forceinline__ int flat_starts(uint32_t *marks, uint32_t off, int items, uint32_t q0,
                                           uint64_t *starts)
{
    const int lane = lane_id();
    lds_u32 *m = lds_ptr(marks);
    if (lane < 2 * N)
        __hip_atomic_store(m + lane, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __builtin_amdgcn_wave_barrier();
    if (lane < items && off >= q0 && off - q0 < WAVE * N)
        __hip_atomic_fetch_or(m + ((off - q0) >> 5), 1u << ((off - q0) & 31u), __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_WORKGROUP);
    __builtin_amdgcn_wave_barrier();
    const uint32_t w = __hip_atomic_load(m + (lane < 2 * N ? lane : 0), __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
    for (int j = 0; j < N; ++j)
        starts[j] = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)w, 2 * j + 1) << 32 |
                    (uint32_t)__builtin_amdgcn_readlane((int)w, 2 * j);
    return __popcll(__ballot(lane < items && off < q0));
}

// The item of this lane's position, given the starts in its 64 positions and
// the number of items that start before them.
__device__ __forceinline__ int flat_item(uint64_t starts, int before)
{
    return before + (int)lanes_below(starts) + (int)((starts >> lane_id()) & 1) - 1;
}

// The lanes with `have` first, in order (a permutation of the wave); the
// lane's new place times 4, for ds_permute.
__device__ __forceinline__ int front_place(uint64_t mask, bool have)
{
    const int below = (int)lanes_below(mask);
    return (have ? below : __popcll(mask) + lane_id() - below) << 2;
}

// Expansion with the arcs of up to 64 queued vertices laid out flat over the
// lanes (the degree-aware mapping of Sec. 3.4 carried to single arcs: every
// lane has an arc whatever the degrees are).  `hubs`: the vertices listed in
// huge_q instead of the queue, the flat arcs of 64 of them at a time dealt out
// over every wave.  Called by whole waves; candidates stay in b until cand_flush.
// Hubs taken one after another cost a chain of four dependent loads each, which
// kept a team (its loads miss the L1 after every barrier) at 4 us a hub.
// Flat, ms before / after: R-MAT scale 17, 1 source 6.5 / 2.0, scale 20, 1
// source 10.7 / 6.2, 48 sources 40.3 / 36.0; one workgroup per source, Kronecker
// scale 16, 256 sources 6.49 / 5.74.  A team's list of 256 was often full, and
// the rest with a wave each: scale 17,
// 16 sources 3.6 / 3.2 with 4096.
template <bool PACKED, int SCOPE, bool BKT = false>
__device__ __forceinline__ void expand_pass(const DevGraph &g, const Slab &S, const ExpandCtx &c,
                                            bool hubs, CandBuf &b, uint32_t &far_min,
                                            uint32_t &outer_min, uint64_t &nimp)
{
    if (c.vw > 0) {
        expand_pass_vw<PACKED, SCOPE, BKT>(g, S, c, c.vw, far_min, outer_min, nimp);
        return;
    }
    const int lane = lane_id();
    constexpr int cap = hub_cap<SCOPE>();
    const int len = hubs             ? (*c.huge_cnt < cap ? *c.huge_cnt : cap)
                    : c.all_vertices ? g.n
                                     : c.len;
    // a short queue is spread over every wave
    int chunk = (len + c.nworkers - 1) / c.nworkers;
    chunk = !hubs && chunk < WAVE ? chunk : WAVE;
    const int first = hubs ? 0 : c.worker * chunk, stride = hubs ? WAVE : c.nworkers * chunk;
    const uint32_t p_first = hubs ? (uint32_t)c.worker * (WAVE * EXPAND_UNROLL) : 0u;
    const uint32_t p_stride = (hubs ? (uint32_t)c.nworkers : 1u) * (WAVE * EXPAND_UNROLL);
    for (int base = first; base < len; base += stride) {
        const int i = base + lane;
        bool valid = lane < chunk && i < len;
        uint32_t beg = 0, end = 0, dv = 0;
        int v = 0;
        if (valid) {
            v = hubs ? c.huge_q[i] : c.all_vertices ? i : c.items[i];
            if (c.all_vertices && !hubs)
                valid = S.stamp[v] == c.cur_tag;
            if (valid) {
                beg = g.row[v];
                end = g.row[v + 1];
                // once per queue entry: the pass that listed a hub cleared its
                // bit, and by now the bit can stand for an entry of next_q
                if (!hubs && v < S.HQ)
                    qbit_clear(S, (uint32_t)v);
                dv = dist_get(S, v);
            }
        }
        uint32_t deg = end - beg;
        if (c.huge_q && !hubs) {
            const bool huge = deg > c.wg_deg;
            const int k = wave_alloc(c.huge_cnt, huge);
            if (huge && k < cap) {
                c.huge_q[k] = v;
                deg = 0;
            }
        }
        // vertices with arcs to the first lanes, in order
        const uint64_t has = __ballot(deg > 0);
        const int items = __popcll(has);
        if (has & (has + 1)) {
            const int dst = front_place(has, deg > 0);
            v = __builtin_amdgcn_ds_permute(dst, v);
            beg = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)beg);
            dv = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)dv);
            deg = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)deg);
        }
        const uint32_t incl = wave_incl_sum_u32(deg);
        const uint32_t off = incl - deg; // strictly increasing over the items
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, WAVE - 1);
        const uint32_t shift = beg - off; // arc position of flat position p: p + shift
        const uint32_t last =
            total - 1u + (uint32_t)__builtin_amdgcn_readlane((int)shift, items > 0 ? items - 1 : 0);
        constexpr int U = EXPAND_UNROLL;
        for (uint32_t p0 = p_first; p0 < total; p0 += p_stride) {
            uint32_t u[U], nd[U], tl[U], wd[U], du[U];
            bool ok[U];
            const int steps = (int)((total - p0 + WAVE - 1) / WAVE); // uniform
            uint64_t starts[U];
            int before = flat_starts<U>(c.marks, off, items, p0, starts);
            // positions past the end read the last arc: no load sits behind a
            // lane's branch, so the steps' loads overlap
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const uint32_t p = p0 + WAVE * j + lane;
                u[j] = nd[j] = tl[j] = wd[j] = du[j] = 0;
                ok[j] = p < total;
                if (j < steps) {
                    const int it = flat_item(starts[j], before);
                    before += __popcll(starts[j]);
                    const uint32_t sh = (uint32_t)__shfl((int)shift, it);
                    nd[j] = (uint32_t)__shfl((int)dv, it);
                    tl[j] = (uint32_t)__shfl(v, it);
                    wd[j] = g.arc[ok[j] ? p + sh : last];
                    if (!PACKED)
                        du[j] = (uint32_t)g.wt[ok[j] ? p + sh : last];
                }
            }
#pragma unroll
            for (int j = 0; j < U; ++j) {
                u[j] = PACKED ? wd[j] >> g.wshift : wd[j];
                nd[j] += PACKED ? (wd[j] & g.wmask) + 1u : du[j];
            }
            dist_peek_n<U>(S, u, nd, ok, du);
#pragma unroll
            for (int j = 0; j < U; ++j)
                ok[j] = ok[j] && nd[j] <= du[j];
            // one copy of the commit code for every j
#pragma nounroll
            for (int j = 0; j < U && j < steps; ++j) {
                cand_add<SCOPE, BKT>(S, c, b, ok[0], u[0], nd[0], tl[0], far_min, outer_min, nimp);
#pragma unroll
                for (int i = 0; i + 1 < U; ++i) {
                    ok[i] = ok[i + 1];
                    u[i] = u[i + 1];
                    nd[i] = nd[i + 1];
                    tl[i] = tl[i + 1];
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Far pile split at a band change.  Entries whose distance dropped below the
// previous threshold were settled through the near queue already (dropped);
// entries below the new threshold move to the near queue and become members
// of the new band; the rest stay in the far pile.  Each vertex sits at most
// once in a pile (it enters when its value first drops into the pile's range).
// ---------------------------------------------------------------------------
struct SplitCtx {
    const int32_t *far_in;
    int len;
    int worker, nworkers;
    uint32_t thr_old, thr;
    int32_t tag;
    int set_tags; // give the moved vertices the queue's tag (node-parallel expansion)
    int32_t *near_q;
    int *near_cnt;
    int32_t *order;
    int *order_cnt;
    int32_t *far_out;
    int *kept_cnt;
};

__device__ __forceinline__ void split_pass(const Slab &S, const SplitCtx &c, uint32_t &kept_min)
{
    const int lane = lane_id();
    for (int base = c.worker * WAVE; base < c.len; base += c.nworkers * WAVE) {
        const int i = base + lane;
        const bool valid = i < c.len;
        int32_t v = 0;
        uint32_t dv = 0;
        if (valid) {
            v = c.far_in[i];
            dv = dist_get(S, v);
        }
        const bool drop = valid && dv < c.thr_old;
        const bool move = valid && !drop && dv < c.thr;
        const bool keep = valid && !drop && !move;
        if (move && v < S.HQ)
            qbit_set(S, (uint32_t)v);
        else if (move && c.set_tags)
            S.stamp[v] = c.tag;
        if (keep)
            kept_min = dv < kept_min ? dv : kept_min;
        int k = wave_alloc(c.near_cnt, move);
        if (move)
            c.near_q[k] = v;
        k = wave_alloc(c.order_cnt, move);
        if (move)
            c.order[k] = v;
        k = wave_alloc(c.kept_cnt, keep);
        if (keep)
            c.far_out[k] = v;
    }
}

// Outer pile pass, when the band threshold has passed the pile bound: entries
// below the old bound went to the inner pile (or a band) when they dropped
// below it and are left out, entries below the new bound join the inner pile,
// the rest stay.
struct OuterSplitCtx {
    const int32_t *outer_in;
    int len;
    int worker, nworkers;
    uint32_t bound_old, bound;
    int32_t *inner_q;
    int *inner_cnt;
    int32_t *outer_out;
    int *kept_cnt;
};

__device__ __forceinline__ void outer_split_pass(const Slab &S, const OuterSplitCtx &c,
                                                 uint32_t &kept_min)
{
    const int lane = lane_id();
    for (int base = c.worker * WAVE; base < c.len; base += c.nworkers * WAVE) {
        const int i = base + lane;
        int32_t v = 0;
        uint32_t dv = 0;
        if (i < c.len) {
            v = c.outer_in[i];
            dv = dist_get(S, v);
        }
        const bool join = i < c.len && dv >= c.bound_old && dv < c.bound;
        const bool keep = i < c.len && dv >= c.bound;
        if (keep)
            kept_min = dv < kept_min ? dv : kept_min;
        int k = wave_alloc(c.inner_cnt, join);
        if (join)
            c.inner_q[k] = v;
        k = wave_alloc(c.kept_cnt, keep);
        if (keep)
            c.outer_out[k] = v;
    }
}

// ---------------------------------------------------------------------------
// Rounds over the members of one band, for the path counts and for the
// dependencies.  A member whose inputs are not all final yet is put on the
// pending list for the next round; the member of least distance among the
// pending ones always has final inputs, so every round makes progress.
// ---------------------------------------------------------------------------
struct RoundCtx {
    const int32_t *items;
    int len;
    int worker, nworkers;
    int lane_max;
    int32_t s;          // the source
    long long src_idx;  // its index in the source list (error reports)
    bool first_round;
    int32_t *pend_q;
    int *pend_cnt;
    unsigned long long *err; // [0] error bits, [1] first overflowing source index
    unsigned int *item_err;  // optional per-source-entry overflow flags
    const int32_t *perm;     // optional: caller's vertex id of each internal vertex
    uint32_t wave_deg;       // more in-arcs than this: the whole wave (else a group of
                             // EXPAND_GROUP lanes above lane_max, one lane below)
};

__device__ __forceinline__ void report_sigma_overflow(unsigned long long *err, long long src_idx,
                                                      unsigned int *item_err)
{
    atomicOr(&err[0], (unsigned long long)BC_ERRBIT_SIGMA);
    atomicMin((long long *)&err[1], src_idx);
    if (item_err)
        item_err[src_idx] = 1u;
}

// Path counts (the counting rule of Alg. 2, evaluated by pulling): sigma[v]
// is the sum of sigma[u] over arcs (u, v, w) with d[u] + w == d[v].  With
// weights >= 1 every such u has d[u] < d[v], so it belongs to this band or
// an earlier one.
template <bool PACKED, int SCOPE>
__device__ __forceinline__ void sigma_round(const DevGraph &g, const Slab &S, const RoundCtx &c, uint64_t &arcs,
                            uint64_t &dag)
{
    const int lane = lane_id();
    for (int base = c.worker * WAVE; base < c.len; base += c.nworkers * WAVE) {
        const int i = base + lane;
        const bool valid = i < c.len;
        int32_t v = 0;
        uint32_t beg = 0, end = 0;
        if (valid) {
            v = c.items[i];
            if (c.first_round)
                arcs += g.row[v + 1] - g.row[v];
        }
        const bool is_src = valid && v == c.s;
        bool pend = false;
        if (valid) {
            beg = g.trow[v];
            end = g.trow[v + 1];
        }
        if (is_src)
            store_f64<SCOPE>(&S.delta[v], -1.0); // sigma[s] = 1 was set at initialisation
        const uint32_t deg = end - beg;
        const bool heavy = valid && !is_src && deg > c.wave_deg;
        const bool mid = valid && !is_src && !heavy && deg > (uint32_t)c.lane_max;
        if (valid && !is_src && !heavy && !mid) {
            const uint32_t dv = dist_get(S, v);
            uint64_t acc = 0;
            bool ready = true, ovf = false;
            uint32_t tight = 0;
            for (uint32_t e0 = beg; e0 < end && ready; e0 += LANE_UNROLL) {
                uint32_t u[LANE_UNROLL], w[LANE_UNROLL], du[LANE_UNROLL];
#pragma unroll
                for (int j = 0; j < LANE_UNROLL; ++j) {
                    u[j] = 0;
                    w[j] = 0;
                    if (e0 + j < end)
                        arc_at<PACKED>(g.tarc, g.twt, e0 + j, g.wshift, g.wmask, u[j], w[j]);
                }
#pragma unroll
                for (int j = 0; j < LANE_UNROLL; ++j)
                    du[j] = e0 + j < end ? dist_get(S, u[j]) : BC_INF;
#pragma unroll
                for (int j = 0; j < LANE_UNROLL; ++j) {
                    if (ready && e0 + j < end && du[j] + w[j] == dv) {
                        const uint64_t su = load_u64<SCOPE>(&S.sigma[u[j]]);
                        if (su == 0) {
                            ready = false;
                        } else {
                            const uint64_t t = acc + su;
                            ovf |= t < acc;
                            acc = t;
                            ++tight;
                        }
                    }
                }
            }
            if (ready) {
                if (ovf) {
                    report_sigma_overflow(c.err, c.src_idx, c.item_err);
                    acc = ~0ull; // stays non-zero so dependants do not wait forever
                }
                store_u64<SCOPE>(&S.sigma[v], acc);
                store_f64<SCOPE>(&S.delta[v], -1.0);
                dag += tight;
            }
            pend = !ready;
        }
        {
            const int k = wave_alloc(c.pend_cnt, pend);
            if (pend)
                c.pend_q[k] = v;
        }
        // Medium in-degree: a group of EXPAND_GROUP lanes per vertex, up to
        // WAVE / EXPAND_GROUP vertices at a time.  Shuffles and ballots run on
        // every lane; each group reads only its own bits.
        uint64_t mm = __ballot(mid);
        const int grp = lane / EXPAND_GROUP, sub = lane % EXPAND_GROUP;
        const int gshift = grp * EXPAND_GROUP;
        const uint64_t gbits = (1ull << EXPAND_GROUP) - 1;
        while (mm) {
            uint64_t t = mm;
            for (int k = 0; k < grp; ++k)
                t &= t - 1;
            const bool have = t != 0;
            const int l = have ? __ffsll((unsigned long long)t) - 1 : 0;
            for (int k = 0; k < WAVE / EXPAND_GROUP; ++k)
                mm &= mm - 1;
            const int32_t mv = __shfl(v, l);
            const uint32_t mb = (uint32_t)__shfl((int)beg, l);
            const uint32_t me0 = (uint32_t)__shfl((int)end, l);
            const uint32_t me = have ? me0 : mb;
            const uint32_t mdv = have ? dist_get(S, mv) : 0u;
            uint64_t acc = 0;
            bool ready = true, ovf = false;
            uint32_t rec = 0; // tight arcs of the group so far (uniform in the group)
            for (uint32_t e0 = mb; e0 < me; e0 += EXPAND_GROUP) {
                const uint32_t e = e0 + sub;
                bool tt = false;
                if (e < me) {
                    uint32_t u, w;
                    arc_at<PACKED>(g.tarc, g.twt, e, g.wshift, g.wmask, u, w);
                    if (dist_get(S, u) + w == mdv) {
                        const uint64_t su = load_u64<SCOPE>(&S.sigma[u]);
                        if (su == 0) {
                            ready = false;
                        } else {
                            const uint64_t x = acc + su;
                            ovf |= x < acc;
                            acc = x;
                            tt = true;
                        }
                    }
                }
                const uint64_t gm = (__ballot(tt) >> gshift) & gbits;
                rec += (uint32_t)__popcll(gm);
                if ((__ballot(!ready) >> gshift) & gbits)
                    break;
            }
            bool gready = ready;
            for (int o = 1; o < EXPAND_GROUP; o <<= 1) {
                const uint64_t y = __shfl_xor(acc, o);
                const int oy = __shfl_xor((int)ovf, o);
                const int ry = __shfl_xor((int)gready, o);
                const uint64_t z = acc + y;
                ovf = ovf || oy || z < acc;
                acc = z;
                gready = gready && ry;
            }
            if (have && gready && sub == 0) {
                if (ovf) {
                    report_sigma_overflow(c.err, c.src_idx, c.item_err);
                    acc = ~0ull;
                }
                store_u64<SCOPE>(&S.sigma[mv], acc);
                store_f64<SCOPE>(&S.delta[mv], -1.0);
                dag += rec;
            }
            const bool p = have && !gready && sub == 0;
            const int k = wave_alloc(c.pend_cnt, p);
            if (p)
                c.pend_q[k] = mv;
        }
        uint64_t hm = __ballot(heavy);
        while (hm) {
            const int l = __ffsll((unsigned long long)hm) - 1;
            hm &= hm - 1;
            const int32_t hv = __shfl(v, l);
            const uint32_t hb = (uint32_t)__shfl((int)beg, l);
            const uint32_t he = (uint32_t)__shfl((int)end, l);
            const uint32_t dv = dist_get(S, hv);
            uint64_t acc = 0;
            bool ready = true, ovf = false;
            uint32_t tight = 0;      // this lane's tight arcs
            for (uint32_t e0 = hb; e0 < he; e0 += WAVE) {
                const uint32_t e = e0 + lane;
                if (e < he) {
                    uint32_t u, w;
                    arc_at<PACKED>(g.tarc, g.twt, e, g.wshift, g.wmask, u, w);
                    if (dist_get(S, u) + w == dv) {
                        const uint64_t su = load_u64<SCOPE>(&S.sigma[u]);
                        if (su == 0) {
                            ready = false;
                        } else {
                            const uint64_t x = acc + su;
                            ovf |= x < acc;
                            acc = x;
                            ++tight;
                        }
                    }
                }
                if (__ballot(!ready))
                    break;
            }
            const bool all_ready = __ballot(!ready) == 0;
            acc = wave_sum_u64_checked(acc, ovf);
            tight = wave_sum_u32(tight);
            if (all_ready && lane == 0) {
                if (ovf) {
                    report_sigma_overflow(c.err, c.src_idx, c.item_err);
                    acc = ~0ull;
                }
                store_u64<SCOPE>(&S.sigma[hv], acc);
                store_f64<SCOPE>(&S.delta[hv], -1.0);
                dag += tight;
            }
            const bool p = !all_ready && lane == 0;
            const int k = wave_alloc(c.pend_cnt, p);
            if (p)
                c.pend_q[k] = hv;
        }
    }
}

// Dependencies (Sec. 2.1 recursion, Alg. 3): delta[v] is the sum over arcs
// (v, u, w) with d[u] == d[v] + w of sigma[v] / sigma[u] * (1 + delta[u]);
// every such u lies in this band or a later one.  A vertex other than the
// source adds its dependency to the centrality (each vertex is one lane's).
template <bool PACKED, int SCOPE>
__device__ __forceinline__ void delta_round(const DevGraph &g, const Slab &S, const RoundCtx &c, double *bc)
{
#pragma clang fp contract(off)
    const int lane = lane_id();
    for (int base = c.worker * WAVE; base < c.len; base += c.nworkers * WAVE) {
        const int i = base + lane;
        const bool valid = i < c.len;
        int32_t v = 0;
        uint32_t beg = 0, end = 0;
        if (valid) {
            v = c.items[i];
            beg = g.row[v];
            end = g.row[v + 1];
        }
        const bool heavy = valid && (end - beg) > (uint32_t)c.lane_max;
        bool pend = false;
        if (valid && !heavy) {
            const uint32_t dv = dist_get(S, v);
            const double sv = (double)S.sigma[v];
            double acc = 0.0;
            bool ready = true;
            for (uint32_t e0 = beg; e0 < end && ready; e0 += LANE_UNROLL) {
                uint32_t u[LANE_UNROLL], w[LANE_UNROLL], du[LANE_UNROLL];
#pragma unroll
                for (int j = 0; j < LANE_UNROLL; ++j) {
                    u[j] = 0;
                    w[j] = 0;
                    if (e0 + j < end)
                        arc_at<PACKED>(g.arc, g.wt, e0 + j, g.wshift, g.wmask, u[j], w[j]);
                }
#pragma unroll
                for (int j = 0; j < LANE_UNROLL; ++j)
                    du[j] = e0 + j < end ? dist_get(S, u[j]) : BC_INF;
#pragma unroll
                for (int j = 0; j < LANE_UNROLL; ++j) {
                    if (ready && du[j] != BC_INF && du[j] == dv + w[j]) {
                        const double dl = load_f64<SCOPE>(&S.delta[u[j]]);
                        if (dl < 0.0)
                            ready = false;
                        else
                            acc += sv / (double)S.sigma[u[j]] * (1.0 + dl);
                    }
                }
            }
            if (ready) {
                store_f64<SCOPE>(&S.delta[v], acc);
                if (v != c.s) {
                    const int32_t o = c.perm ? c.perm[v] : v;
                    bc[o] += acc;
                }
            }
            pend = !ready;
        }
        {
            const int k = wave_alloc(c.pend_cnt, pend);
            if (pend)
                c.pend_q[k] = v;
        }
        uint64_t hm = __ballot(heavy);
        while (hm) {
            const int l = __ffsll((unsigned long long)hm) - 1;
            hm &= hm - 1;
            const int32_t hv = __shfl(v, l);
            const uint32_t hb = (uint32_t)__shfl((int)beg, l);
            const uint32_t he = (uint32_t)__shfl((int)end, l);
            const uint32_t dv = dist_get(S, hv);
            const double sv = (double)S.sigma[hv];
            double acc = 0.0;
            bool ready = true;
            for (uint32_t e = hb + lane; e < he; e += WAVE) {
                uint32_t u, w;
                arc_at<PACKED>(g.arc, g.wt, e, g.wshift, g.wmask, u, w);
                const uint32_t du = dist_get(S, u);
                if (du != BC_INF && du == dv + w) {
                    const double dl = load_f64<SCOPE>(&S.delta[u]);
                    if (dl < 0.0) {
                        ready = false;
                        break;
                    }
                    acc += sv / (double)S.sigma[u] * (1.0 + dl);
                }
            }
            const bool all_ready = __ballot(!ready) == 0;
            acc = wave_sum_f64(acc);
            if (all_ready && lane == 0) {
                store_f64<SCOPE>(&S.delta[hv], acc);
                if (hv != c.s) {
                    const int32_t o = c.perm ? c.perm[hv] : hv;
                    bc[o] += acc;
                }
            }
            const bool p = !all_ready && lane == 0;
            const int k = wave_alloc(c.pend_cnt, p);
            if (p)
                c.pend_q[k] = hv;
        }
    }
}

// ---------------------------------------------------------------------------
// Batched form: path counts and dependencies by levels of the shortest-path
// DAG.
//
// A band's members are counted in rounds; a member is final in the first
// round that finds all its DAG predecessors final in earlier rounds.  Its
// record then holds that round's number, which only grows over the slab's
// life, so a predecessor is final exactly when its number lies between the
// source's first and the current one: one finished in the current round
// reads as pending whichever of the two its reader sees, and no order
// between its fields matters.  The vertices of a round form a level: no DAG
// arc lies inside it.  Levels are appended to order[] one after another, and
// the dependency pass walks them backwards (Alg. 3): every level adds its
// terms into its predecessors, and needs neither successor counts nor
// queues.  Per DAG arc that leaves one atomic; successor counts took two more,
// and a flag or bucket atomic per improvement went with the piles' entries
// following from the replaced distance (relax_commit).  Scattered global
// atomics are what bounds the kernel: 256 workgroups of 1024 threads reach
// 27 to 31 G/s of them while each stays within 0.8 MB, 18 to 20 G/s beyond,
// returning or not, 32 or 64 bits, against 50 to 300 G/s for loads; with 7.7
// per reached vertex a Barabasi-Albert run spent about 160 of its 197 ms at
// that rate.  Barabasi-Albert n = 100,000, 4096 sources: 169 -> 129 ms; R-MAT
// scale 20, 1024 sources: 311 -> 261 ms; 1000 x 1000 grid, 256 sources: 108 ->
// 86 ms (flat expansion with candidate batches -> levels).
//
// Predecessors of v, once known (d[v] is final): pred1 >= 0 is the only one;
// -(m + 1) says that preds[trow[v] ..] lists m of them, as tails, or as
// in-row positions when edge betweenness is asked for; -1: none (the source).
// ---------------------------------------------------------------------------
struct CountCtx {
    const int32_t *items;
    int len;
    int worker, nworkers;
    uint32_t *marks;      // 2 words of LDS of this wave
    int lane_max;         // lists up to this long are summed by one lane, longer by the wave
    long long src_idx;    // index in the source list (error reports)
    int32_t base, cur;    // round numbers: the source's own level, this round
    int32_t *fin_q;       // vertices final in this round
    int *fin_cnt;
    int32_t *pend_q;      // vertices for the next round
    int *pend_cnt;
    unsigned long long *err;
    unsigned int *item_err;
    int keys;             // predecessor keys were recorded
    int positions;        // lists hold in-row positions (edge betweenness)
};

// A recorded predecessor: the tail of the in-arc at in-row position pos.
template <bool PACKED>
__device__ __forceinline__ int32_t pred_vertex(const DevGraph &g, int32_t pos)
{
    uint32_t u, w;
    arc_at<PACKED>(g.tarc, g.twt, (uint32_t)pos, g.wshift, g.wmask, u, w);
    return (int32_t)u;
}

// Sum of the counts of the m predecessors listed at preds[b] onwards, over
// the list entries first, first + step, ...; ready turns false when one is
// not final yet.
template <bool PACKED>
__device__ __forceinline__ void list_sum(const DevGraph &g, const Slab &S, const CountCtx &c,
                                         uint32_t b, uint32_t m, uint32_t first, uint32_t step,
                                         uint64_t &acc, bool &ready, bool &ovf)
{
    for (uint32_t j = first; j < m && ready; j += step) {
        int32_t u = S.preds[b + j];
        if (c.positions)
            u = pred_vertex<PACKED>(g, u);
        const uint32_t lv = (uint32_t)(S.level[u] - c.base);
        const uint64_t su = S.sigma[u];
        if (lv < (uint32_t)(c.cur - c.base)) {
            const uint64_t x = acc + su;
            ovf |= x < acc;
            acc = x;
        } else {
            ready = false;
        }
    }
}

template <bool PACKED, int SCOPE>
__device__ __forceinline__ void count_pass(const DevGraph &g, const Slab &S, const CountCtx &c,
                                           uint64_t &dag)
{
    const int lane = lane_id();
    int chunk = (c.len + c.nworkers - 1) / c.nworkers;
    chunk = chunk < WAVE ? chunk : WAVE;
    for (int base = c.worker * chunk; base < c.len; base += c.nworkers * chunk) {
        const int i = base + lane;
        const bool valid = lane < chunk && i < c.len;
        int32_t v = 0, p1 = -1;
        uint32_t tb = 0, te = 0;
        bool scan = false;
        if (valid) {
            v = c.items[i];
            const uint64_t key = *key_ptr(S, v);
            const int32_t fl = S.flags[v];
            const uint32_t nt = (uint32_t)fl >> TIE_SHIFT;
            // a resident vertex's key is the last one stored: of the final
            // distance, but for a race between two improvements
            const bool keyed = c.keys && key != KEY_NONE &&
                               (v >= S.H || (uint32_t)(key >> 32) == dist_get(S, (uint32_t)v));
            if (fl & VFLAG_LIST) {
                p1 = S.pred1[v];
                if (p1 < 0)
                    tb = g.trow[v];
            } else if (keyed && nt == 0) {
                p1 = (int32_t)(uint32_t)key; // the key's tail alone
            } else {
                tb = g.trow[v];
                te = g.trow[v + 1];
                scan = true;
                if (keyed && nt <= TIE_MAX && tb + 2 * nt <= te) {
                    // The pairs at the key's distance name the other tails.  The
                    // list grows over the pairs from the front: entry j <= i + 1 is
                    // written after pair i (slots 2i, 2i + 1) was read.
                    const uint32_t dk = (uint32_t)(key >> 32);
                    const int32_t u0 = (int32_t)(uint32_t)key;
                    uint32_t m = 1;
                    bool twice = false;
                    for (uint32_t k = 0; k < nt && !twice; ++k) {
                        const uint32_t dk2 = (uint32_t)S.preds[tb + 2 * k];
                        const int32_t t = S.preds[tb + 2 * k + 1];
                        if (dk2 != dk)
                            continue;
                        twice = t == u0;
                        for (uint32_t j = 1; j < m; ++j)
                            twice |= S.preds[tb + j] == t;
                        S.preds[tb + m] = t;
                        ++m;
                    }
                    if (!twice) { // else a tail is seen twice: scan
                        scan = false;
                        if (m == 1) {
                            p1 = u0;
                        } else {
                            S.preds[tb] = u0;
                            p1 = -(int32_t)(m + 1);
                        }
                        S.pred1[v] = p1;
                        S.flags[v] = fl | VFLAG_LIST;
                    }
                }
            }
        }
        // The others test their in-arcs, laid out flat over the lanes, and list
        // the tight ones.
        const uint64_t sm = __ballot(scan);
        if (sm) {
            const int items = __popcll(sm);
            const int dst = front_place(sm, scan);
            const int32_t sv = __builtin_amdgcn_ds_permute(dst, v);
            const uint32_t sb = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)tb);
            const uint32_t se = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)te);
            const bool mine = lane < items;
            const uint32_t sd = mine ? dist_get(S, sv) : 0u;
            const uint32_t deg = mine ? se - sb : 0u;
            const uint32_t incl = wave_incl_sum_u32(deg);
            const uint32_t off = incl - deg;
            const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, WAVE - 1);
            uint32_t m = 0; // tight arcs of the lane's item so far
            for (uint32_t q0 = 0; q0 < total; q0 += WAVE) {
                uint64_t starts;
                const int before = flat_starts<1>(c.marks, off, items, q0, &starts);
                const int it = flat_item(starts, before);
                const uint32_t p = q0 + lane;
                const uint32_t ib = (uint32_t)__shfl((int)sb, it);
                const uint32_t io = (uint32_t)__shfl((int)off, it);
                const uint32_t id = (uint32_t)__shfl((int)sd, it);
                const uint32_t im = (uint32_t)__shfl((int)m, it);
                bool tight = false;
                uint32_t u = 0, w = 0;
                if (p < total) {
                    arc_at<PACKED>(g.tarc, g.twt, ib + (p - io), g.wshift, g.wmask, u, w);
                    tight = dist_get(S, u) + w == id;
                }
                const uint64_t tm = __ballot(tight);
                // the item's lanes start at flat position io (or earlier than q0)
                const uint32_t lo = io > q0 ? io - q0 : 0u;
                if (tight)
                    S.preds[ib + im + __popcll(tm & ((1ull << lane) - (1ull << lo)))] =
                        c.positions ? (int32_t)(ib + (p - io)) : (int32_t)u;
                if (mine && off < q0 + WAVE && off + deg > q0) {
                    const uint32_t a = off > q0 ? off - q0 : 0u;
                    const uint32_t z = off + deg - q0;
                    const uint64_t upto = z >= WAVE ? ~0ull : (1ull << z) - 1;
                    m += (uint32_t)__popcll(tm & upto & ~((1ull << a) - 1));
                }
            }
            // the lists were written by other lanes of this wave
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const uint32_t mm = (uint32_t)__shfl((int)m, dst >> 2);
            if (scan) {
                p1 = mm == 1 && !c.positions ? S.preds[tb] : -(int32_t)(mm + 1);
                S.pred1[v] = p1;
                S.flags[v] = VFLAG_LIST | (S.flags[v] & VFLAG_OUTER);
            }
        }
        uint64_t acc = 0;
        bool ready = false, ovf = false;
        uint32_t m = 0;
        bool wide = false;
        if (valid && p1 >= 0) {
            const uint32_t lv = (uint32_t)(S.level[p1] - c.base);
            acc = S.sigma[p1];
            ready = lv < (uint32_t)(c.cur - c.base);
            m = 1;
        } else if (valid) {
            m = (uint32_t)(-p1 - 1);
            wide = m > (uint32_t)c.lane_max;
            ready = m > 0;
            if (!wide)
                list_sum<PACKED>(g, S, c, tb, m, 0, 1, acc, ready, ovf);
        }
        uint64_t hm = __ballot(wide);
        while (hm) {
            const int l = __ffsll((unsigned long long)hm) - 1;
            hm &= hm - 1;
            const uint32_t hb = (uint32_t)__shfl((int)tb, l);
            const uint32_t hn = (uint32_t)__shfl((int)m, l);
            uint64_t x = 0;
            bool r = true, o = false;
            list_sum<PACKED>(g, S, c, hb, hn, (uint32_t)lane, WAVE, x, r, o);
            const bool all = __ballot(!r) == 0;
            x = wave_sum_u64_checked(x, o);
            if (lane == l) {
                acc = x;
                ready = all;
                ovf = o;
            }
        }
        if (valid && ready) {
            if (ovf) {
                report_sigma_overflow(c.err, c.src_idx, c.item_err);
                acc = ~0ull;
            }
            S.level[v] = c.cur;
            S.pred1[v] = p1;
            S.sigma[v] = acc;
            S.delta[v] = 0.0;
            dag += m;
        }
        int k = wave_alloc(c.fin_cnt, valid && ready);
        if (valid && ready)
            c.fin_q[k] = v;
        k = wave_alloc(c.pend_cnt, valid && !ready);
        if (valid && !ready)
            c.pend_q[k] = v;
    }
}

// One level's dependencies (Sec. 2.1 recursion, Alg. 3): every member w is
// final and adds sigma[u] / sigma[w] * (1 + delta[w]) into each recorded
// predecessor u.
struct PushCtx {
    const int32_t *items;
    int len;
    int worker, nworkers;
    uint32_t *marks;      // 2 words of LDS of this wave
    double *ebc;          // optional edge betweenness (caller arc order; lists hold positions)
    const uint32_t *emap; // in-row position -> caller arc index
};

template <bool PACKED, int SCOPE>
__device__ __forceinline__ void push_level(const DevGraph &g, const Slab &S, const PushCtx &c)
{
#pragma clang fp contract(off)
    const int lane = lane_id();
    int chunk = (c.len + c.nworkers - 1) / c.nworkers;
    chunk = chunk < WAVE ? chunk : WAVE;
    for (int base = c.worker * chunk; base < c.len; base += c.nworkers * chunk) {
        const int i = base + lane;
        const bool valid = lane < chunk && i < c.len;
        int32_t w = 0, p1 = -1;
        double dw = 0.0;
        if (valid) {
            w = c.items[i];
            p1 = S.pred1[w];
            dw = S.delta[w];
        }
        // the only predecessor's count was copied: the ratio is exactly 1
        if (valid && p1 >= 0)
            __hip_atomic_fetch_add(&S.delta[p1], 1.0 + dw, __ATOMIC_RELAXED, SCOPE);
        const bool list = valid && p1 < -1;
        const uint64_t lm = __ballot(list);
        if (lm) {
            uint32_t tb = 0;
            double sw = 1.0;
            if (list) {
                tb = g.trow[w];
                sw = (double)S.sigma[w];
            }
            const int items = __popcll(lm);
            const int dst = front_place(lm, list);
            const uint32_t sb = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)tb);
            const int from = __builtin_amdgcn_ds_permute(dst, lane);
            const int fp = __shfl(p1, from);
            const uint32_t deg = lane < items ? (uint32_t)(-fp - 1) : 0u;
            const uint32_t incl = wave_incl_sum_u32(deg);
            const uint32_t off = incl - deg;
            const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, WAVE - 1);
            const uint32_t shift = sb - off;
            for (uint32_t q0 = 0; q0 < total; q0 += WAVE) {
                uint64_t starts;
                const int before = flat_starts<1>(c.marks, off, items, q0, &starts);
                const int it = flat_item(starts, before);
                const uint32_t p = q0 + lane;
                const uint32_t sh = (uint32_t)__shfl((int)shift, it);
                const int src = __shfl(from, it);
                const double hd = __shfl(dw, src);
                const double hs = __shfl(sw, src);
                if (p < total) {
                    const int32_t e = S.preds[p + sh];
                    const int32_t u = c.ebc ? pred_vertex<PACKED>(g, e) : e;
                    const double term = (double)S.sigma[u] / hs * (1.0 + hd);
                    if (c.ebc) // the term is the source's dependency on the arc u -> w
                        unsafeAtomicAdd(&c.ebc[c.emap[e]], term);
                    __hip_atomic_fetch_add(&S.delta[u], term, __ATOMIC_RELAXED, SCOPE);
                }
            }
        }
    }
}

// One level's dependencies by pulling over the out-arcs: every successor lies
// in a later level, whose dependencies are final.
template <bool PACKED>
__device__ __forceinline__ void pull_level(const DevGraph &g, const Slab &S, const int32_t *items,
                                           int len, int worker, int nworkers, int lane_max)
{
#pragma clang fp contract(off)
    const int lane = lane_id();
    for (int base = worker * WAVE; base < len; base += nworkers * WAVE) {
        const int i = base + lane;
        const bool valid = i < len;
        int32_t v = 0;
        uint32_t beg = 0, end = 0;
        if (valid) {
            v = items[i];
            beg = g.row[v];
            end = g.row[v + 1];
        }
        const bool heavy = valid && end - beg > (uint32_t)lane_max;
        auto term = [&](uint32_t e, uint32_t dv, double sv) {
            uint32_t u, w;
            arc_at<PACKED>(g.arc, g.wt, e, g.wshift, g.wmask, u, w);
            const uint32_t du = dist_get(S, u);
            return du != BC_INF && du == dv + w ? sv / (double)S.sigma[u] * (1.0 + S.delta[u])
                                                : 0.0;
        };
        if (valid && !heavy) {
            const uint32_t dv = dist_get(S, v);
            const double sv = (double)S.sigma[v];
            double acc = 0.0;
            for (uint32_t e = beg; e < end; ++e)
                acc += term(e, dv, sv);
            S.delta[v] = acc;
        }
        uint64_t hm = __ballot(heavy);
        while (hm) {
            const int l = __ffsll((unsigned long long)hm) - 1;
            hm &= hm - 1;
            const int32_t hv = __shfl(v, l);
            const uint32_t hb = (uint32_t)__shfl((int)beg, l);
            const uint32_t he = (uint32_t)__shfl((int)end, l);
            const uint32_t dv = dist_get(S, hv);
            const double sv = (double)S.sigma[hv];
            double acc = 0.0;
            for (uint32_t e = hb + lane; e < he; e += WAVE)
                acc += term(e, dv, sv);
            acc = wave_sum_f64(acc);
            if (lane == 0)
                S.delta[hv] = acc;
        }
    }
}
