// team.hip -- the batched form with several workgroups per source, for source
// lists that are shorter than the GPU has compute units.
//
// One workgroup per source leaves the other CUs idle, and a large graph's
// source then takes as long as one CU's share of scattered accesses allows.
// Here a team of workgroups shares one source and one state slab: the same
// passes (passes.h) run over all waves of the team, with the counters in
// global memory, agent scope, and a barrier of the team between steps.
// Distances all live in the slab (the workgroups cannot see each other's LDS);
// each workgroup keeps upper bounds of those of the highest in-degrees in its
// LDS, a byte each, which answer most of the expansion's checks.  Without them
// the expansion ran at the rate of random reads of d[] (50 G/s), R-MAT scale 20:
// 16 sources 14.0 -> 12.4 ms, 48 sources 34.3 -> 27.7 ms, 64 sources 41.9 -> 34.3
// ms; Barabasi-Albert 1M, 48 sources 31.4 -> 30.2, 1 source 5.05 / 5.1.
//
// Teams form as workgroups start: a workgroup joins the first team that is
// still open, the first member closes its team once it is full or after
// TEAM_JOIN_TICKS, and only members that joined are waited for, so that no
// wait depends on a workgroup that has not started.  A workgroup that finds
// every team closed leaves.  Teams take sources from the device counter until
// none is left, however many teams formed.
#include "kernels.h"
#include "dev_common.h"
#include "passes.h"

#define AG_SCOPE __HIP_MEMORY_SCOPE_AGENT

#define TEAM_CLOSED 0x80000000u
#define TEAM_JOIN_TICKS 2000ll          // 20 us of the 100 MHz device clock

extern __shared__ uint32_t seen_bounds[];

static_assert(TEAM_HUBS == EXPAND_TEAM_CAP, "the hub list of a pass");

template <class T> __device__ __forceinline__ T ag_load(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, AG_SCOPE);
}

template <class T> __device__ __forceinline__ void ag_store(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, AG_SCOPE);
}

// One workgroup's view of its team.  Every member runs the same control flow
// on the same values, read after each barrier.
struct TeamWg {
    uint32_t marks[TEAM_THREADS / WAVE][2 * EXPAND_UNROLL];
    int team, rank, members, failed;
    // after a barrier: what the interval appended, and the band's far pile
    // (words that the next interval may change are never read after a barrier:
    // a slow member would see another value than a fast one)
    int step[TEAM_STEP_WORDS];
    int far_cnt;
    uint32_t far_min;
    long long src;
};
static_assert(sizeof(TeamWg) <= TEAM_LDS_CTL, "the bounds leave room for TeamWg");

struct TeamSync {
    TeamCtl *ctl;
    unsigned int epoch; // arrivals that complete the next barrier (thread 0)
    int interval;       // barrier intervals so far, mod 3
    unsigned int looks; // looks at a barrier before it has failed
};

// Barrier of the team.  The release before and the acquire after it (of thread
// 0, between workgroup barriers) order every member's accesses; a barrier
// costs 1.7 us for a team of 2 to 8 alone on the GPU, 8 us when 256 workgroups
// are in barriers at once.  All members run and none leaves early, so each wait
// ends; the bound is there for the case that this is not so.  It counts looks,
// not time: on a GPU shared with other processes a team is slow while it is off
// the GPU, and then all of it is.  A member that sees a failure, its own or
// another's, reports it itself at the end: the first member may be the one that came
// late and sees its barriers complete, and its next one can be that of a new source.
// `par`, `band`: which of the source and far pile words to read.
__device__ __forceinline__ bool team_barrier(TeamWg &W, TeamSync &y, int par, int band)
{
    // every wave's stores have reached the L2 before thread 0 releases them (a
    // workgroup barrier alone does not wait for them)
    __builtin_amdgcn_s_waitcnt(0x0f70); // vmcnt(0)
    __syncthreads();
    if (threadIdx.x == 0) {
        TeamCtl *c = y.ctl;
        const int nx = y.interval == 2 ? 0 : y.interval + 1;
        if (W.rank == 0) // last read after the barrier before the previous one
            for (int i = 0; i < TEAM_STEP_WORDS; ++i)
                ag_store(&c->step[nx][i], 0);
        y.epoch += (unsigned int)W.members;
        __threadfence();
        __hip_atomic_fetch_add(&c->arrived, 1u, __ATOMIC_RELAXED, AG_SCOPE);
        for (unsigned int looks = 0; (int)(ag_load(&c->arrived) - y.epoch) < 0;) {
            __builtin_amdgcn_s_sleep(1);
            const bool late = ++looks >= y.looks;
            if (late)
                ag_store(&c->failed, 1u);
            if ((late || (looks & 1023u) == 0u) && ag_load(&c->failed)) {
                W.failed = 1;
                break;
            }
        }
        __threadfence();
        for (int i = 0; i < TEAM_STEP_WORDS; ++i)
            W.step[i] = ag_load(&c->step[y.interval][i]);
        W.far_cnt = ag_load(&c->far_cnt[band]);
        W.far_min = ag_load(&c->far_min[band]);
        W.src = ag_load(&c->src[par]);
    }
    y.interval = y.interval == 2 ? 0 : y.interval + 1;
    __syncthreads();
    return W.failed == 0;
}

template <bool PACKED>
__global__ __launch_bounds__(TEAM_THREADS, 4) void k_team(TeamArgs ta)
{
    __shared__ TeamWg W;
    const BatchArgs &a = ta.b;
    const int tid = threadIdx.x;
    const DevGraph &g = a.g;
    const int n = g.n;
    TeamSync y{nullptr, 0u, 0, ta.looks};
    if (tid == 0) {
        W.failed = 0;
        W.team = -1;
        // Consecutive workgroups start on the eight XCDs in turn, and a team inside
        // one shares its L2: class c holds the teams c, c + 8, ..., and a workgroup
        // asks the teams class by class, from its own class on.  (blockIdx + i) mod
        // teams / this, ms: R-MAT scale 20, 7 sources 10.3 / 7.7, 9 sources
        // 11.5 / 9.1; Barabasi-Albert 1M, 7 sources 10.2 / 8.5; ER 500k, 17 sources 7.7
        // / 7.0; 8 and 16 teams, in their classes either way, the same.
        const int classes = ta.teams < 8 ? ta.teams : 8;
        const int q = ta.teams / classes, more = ta.teams % classes; // the first have q + 1
        const int own = (int)(blockIdx.x % 8u) % classes;
        const int at = own * q + (own < more ? own : more) +
                       (int)(blockIdx.x / 8u) % (own < more ? q + 1 : q);
        for (int i = 0; i < ta.teams && W.team < 0; ++i) {
            const int x = (at + i) % ta.teams, y = x - more * (q + 1);
            const int t = y < 0 ? x / (q + 1) + classes * (x % (q + 1))
                                : more + y / q + classes * (y % q);
            TeamCtl *c = &ta.ctl[t];
            if (ag_load(&c->joined) >= (unsigned)ta.size) // full or closed
                continue;
            const unsigned int r = __hip_atomic_fetch_add(&c->joined, 1u, __ATOMIC_RELAXED,
                                                          AG_SCOPE);
            if ((r & TEAM_CLOSED) || r >= (unsigned)ta.size)
                continue;
            W.team = t;
            W.rank = (int)r;
            if (r == 0) {
                const long long t0 = wall_clock64();
                while (ag_load(&c->joined) < (unsigned)ta.size &&
                       wall_clock64() - t0 < TEAM_JOIN_TICKS)
                    __builtin_amdgcn_s_sleep(1);
                const unsigned int m = __hip_atomic_fetch_or(&c->joined, TEAM_CLOSED,
                                                             __ATOMIC_RELAXED, AG_SCOPE);
                W.members = (int)(m < (unsigned)ta.size ? m : (unsigned)ta.size);
                ag_store(&c->members, (unsigned int)W.members);
            } else { // the first member is running and closes the team soon
                unsigned int m;
                while ((m = ag_load(&c->members)) == 0u)
                    __builtin_amdgcn_s_sleep(1);
                W.members = (int)m;
            }
        }
    }
    __syncthreads();
    if (W.team < 0)
        return;
    TeamCtl *const c = &ta.ctl[W.team];
    y.ctl = c;
    const int rank = W.rank, members = W.members;
    const bool lead = rank == 0 && tid == 0;
    const int gtid = rank * TEAM_THREADS + tid, gn = members * TEAM_THREADS;
    const int worker = __builtin_amdgcn_readfirstlane(rank * (TEAM_THREADS / WAVE) + wave_index());
    const int nworkers = members * (TEAM_THREADS / WAVE);
    uint32_t *const marks = W.marks[wave_index()];
    Slab S = slab_at(a.slab_base, a.L, W.team);
    S.seen = seen_bounds;
    S.HB = ta.bounds;
    S.bshift = ta.bshift;
    lds_u32 *const bounds = lds_ptr(seen_bounds);
    const int bound_words = ta.bounds / 4;
    int32_t gen = (int32_t)S.hdr[0], lvl = (int32_t)S.hdr[1];
    uint64_t st_arcs = 0, st_dag = 0, st_imp = 0;
    const unsigned long long iter_cap = 8ull * (unsigned long long)n + 1024ull;
    unsigned long long ticks[5] = {0, 0, 0, 0, 0}, srounds = 0, drounds = 0;
    long long tmark = lead ? wall_clock64() : 0;
    auto mark = [&](int phase) {
        if (lead) {
            const long long t = wall_clock64();
            ticks[phase] += (unsigned long long)(t - tmark);
            tmark = t;
        }
    };

    bool alive = true;
    for (int par = 0; alive; par ^= 1) {
        if (lead)
            ag_store(&c->src[par], (long long)__hip_atomic_fetch_add(a.next_src, 1ull,
                                                                     __ATOMIC_RELAXED, AG_SCOPE));
        if (!(alive = team_barrier(W, y, par, 0)))
            break;
        const long long idx = W.src;
        if (idx >= a.k)
            break;
        const int32_t s_in = a.sources[idx];
        if (s_in < 0 || s_in >= n) {
            if (lead)
                atomicOr(&a.err[0], (unsigned long long)BC_ERRBIT_SOURCE);
            continue;
        }
        const int32_t s = a.iperm ? a.iperm[s_in] : s_in;
        const bool restart = gen > (1 << 30) || lvl > (1 << 30); // long before they wrap
        if (restart)
            gen = lvl = 0;
        gen += 1;
        lvl += 1;
        const int32_t base = lvl;
        for (int v = gtid; v < n; v += gn) {
            const bool is = v == s; // final from the start, a level of its own
            S.d[v] = is ? 0u : BC_INF;
            *key_ptr(S, v) = is ? 0ull : KEY_NONE; // the source's dependency is 0.0
            S.flags[v] = 0;
            S.stamp[v] = 0;
            if (restart)
                S.level[v] = 0;
            if (is) {
                S.level[v] = base;
                S.pred1[v] = -1;
                S.sigma[v] = 1;
            }
        }
        S.base8 = 0;
        for (int i = tid; i < bound_words; i += TEAM_THREADS)
            bounds[i] = ~0u;
        if (lead) {
            S.qa[0] = s;
            S.order[0] = s;
            S.band_off[0] = 0;
            S.band_off[1] = 1;
            for (int i = 0; i < 2; ++i) {
                ag_store(&c->far_cnt[i], 0);
                ag_store(&c->far_min[i], BC_INF);
            }
        }
        int band = 0, cur = 0, fcur = 0, near_len = 1, nlev = 1, nbands = 0;
        int band_start = 1, total = 1; // members before this band, and so far
        uint32_t thr = a.delta;
        unsigned long long iters = 0;
        bool ok = team_barrier(W, y, par, band);
        mark(0);

        while (ok) {
            while (ok && near_len > 0) {
                ExpandCtx ec;
                ec.items = cur ? S.qb : S.qa;
                ec.len = near_len;
                ec.all_vertices = 0;
                ec.cur_tag = gen;
                ec.vw = 0;
                ec.worker = worker;
                ec.nworkers = nworkers;
                ec.marks = marks;
                ec.thr = thr;
                ec.tag_next = gen + 1;
                ec.next_q = cur ? S.qa : S.qb;
                ec.next_cnt = &c->step[y.interval][TEAM_NEAR];
                ec.order = S.order + total;
                ec.order_cnt = &c->step[y.interval][TEAM_MEMBER];
                ec.far_q = fcur ? S.fb : S.fa;
                ec.far_cnt = &c->far_cnt[band];
                ec.bound = BC_INF; // one far pile: the whole team scans it
                ec.outer_q = nullptr;
                ec.outer_cnt = nullptr;
                ec.huge_q = a.hubs ? c->hub_q : nullptr;
                ec.huge_cnt = &c->step[y.interval][TEAM_HUB];
                ec.keys = a.ebc == nullptr;
                ec.trow = g.trow;
                ec.wg_deg = a.wg_deg;
                ec.bk = nullptr;
                uint32_t fmin = BC_INF, omin = BC_INF;
                CandBuf cb{0u, 0u, 0u, 0};
#pragma nounroll
                for (int part = 0;; ++part) {
                    expand_pass<PACKED, AG_SCOPE>(g, S, ec, part == 1, cb, fmin, omin, st_imp);
                    cand_flush<AG_SCOPE, false>(S, ec, cb, fmin, omin, st_imp);
                    fmin = wave_min_u32(fmin);
                    if (lane_id() == 0 && fmin != BC_INF)
                        atomicMin(&c->far_min[band], fmin);
                    fmin = BC_INF;
                    ok = team_barrier(W, y, par, band);
                    near_len = part == 0 ? W.step[TEAM_NEAR] : near_len + W.step[TEAM_NEAR];
                    total += W.step[TEAM_MEMBER];
                    if (!ok || part == 1 || W.step[TEAM_HUB] == 0)
                        break;
                    // the listed hubs, spread over the whole team (huge_cnt keeps
                    // naming the closed interval's word)
                    ec.next_q += near_len;
                    ec.next_cnt = &c->step[y.interval][TEAM_NEAR];
                    ec.order = S.order + total;
                    ec.order_cnt = &c->step[y.interval][TEAM_MEMBER];
                }
                cur ^= 1;
                gen += 1;
                if (++iters > iter_cap)
                    ok = false;
            }
            mark(1);
            if (!ok)
                break;
            // the band is closed: count its members level by level
            const int b0 = band_start, b1 = total;
            const int far_len = W.far_cnt;
            const uint32_t far_min = W.far_min;
            if (b1 > b0) {
                const int32_t *items = S.order + b0;
                int len = b1 - b0, done = 0, first = 0;
                for (int round = 0; ok; ++round) {
                    lvl += 1;
                    CountCtx cc;
                    cc.items = items;
                    cc.len = len;
                    cc.worker = worker;
                    cc.nworkers = nworkers;
                    cc.marks = marks;
                    cc.lane_max = a.lane_max;
                    cc.src_idx = idx;
                    cc.base = base;
                    cc.cur = lvl;
                    cc.fin_q = round == 0 ? S.oa : S.order + b0 + done;
                    cc.fin_cnt = &c->step[y.interval][TEAM_FINAL];
                    cc.pend_q = round & 1 ? S.qb : S.qa;
                    cc.pend_cnt = &c->step[y.interval][TEAM_PEND];
                    cc.err = a.err;
                    cc.item_err = a.item_err;
                    cc.keys = a.ebc == nullptr;
                    cc.positions = a.ebc != nullptr;
                    if (round == 1) // over the members that the first round read
                        for (int i = gtid; i < first; i += gn)
                            S.order[b0 + i] = S.oa[i];
                    count_pass<PACKED, AG_SCOPE>(g, S, cc, st_dag);
                    if (!(ok = team_barrier(W, y, par, band)))
                        break;
                    const int np = W.step[TEAM_PEND], nf = W.step[TEAM_FINAL];
                    if (round == 0)
                        first = nf;
                    done += nf;
                    nlev += 1;
                    srounds += 1;
                    if (lead)
                        S.band_off[nlev] = b0 + done;
                    if (np == 0)
                        break;
                    ok = nf > 0;
                    items = cc.pend_q;
                    len = np;
                }
                nbands += 1;
            }
            band_start = b1;
            mark(2);
            if (!ok || far_len == 0)
                break;
            // next band: threshold from the least far distance seen
            const uint32_t thr_old = thr;
            thr = sat_add_u32(far_min > thr ? far_min : thr, (uint64_t)a.delta);
            gen += 1;
            const int nb = band == 2 ? 0 : band + 1, nnb = nb == 2 ? 0 : nb + 1;
            if (lead) { // last read before the previous band
                ag_store(&c->far_cnt[nnb], 0);
                ag_store(&c->far_min[nnb], BC_INF);
            }
            SplitCtx sp;
            sp.far_in = fcur ? S.fb : S.fa;
            sp.len = far_len;
            sp.worker = worker;
            sp.nworkers = nworkers;
            sp.thr_old = thr_old;
            sp.thr = thr;
            sp.tag = gen;
            sp.set_tags = 0;
            sp.near_q = cur ? S.qb : S.qa;
            sp.near_cnt = &c->step[y.interval][TEAM_NEAR];
            sp.order = S.order + total;
            sp.order_cnt = &c->step[y.interval][TEAM_MEMBER];
            sp.far_out = fcur ? S.fa : S.fb;
            sp.kept_cnt = &c->far_cnt[nb];
            const uint32_t up = (thr_old - S.base8) >> S.bshift;
            if (up >= SEEN_REBASE) { // every offer from here on is above thr_old
                S.base8 += up << S.bshift;
                for (int i = tid; i < bound_words; i += TEAM_THREADS) {
                    const uint32_t x = bounds[i];
                    uint32_t y = 0;
#pragma unroll
                    for (int b = 0; b < 32; b += 8) {
                        const uint32_t e = (x >> b) & 0xffu;
                        y |= (e == SEEN_NONE ? e : e > up ? e - up : 0u) << b;
                    }
                    bounds[i] = y;
                }
            }
            uint32_t kmin = BC_INF;
            split_pass(S, sp, kmin);
            kmin = wave_min_u32(kmin);
            if (lane_id() == 0 && kmin != BC_INF)
                atomicMin(&c->far_min[nb], kmin);
            fcur ^= 1;
            band = nb;
            ok = team_barrier(W, y, par, band);
            near_len = W.step[TEAM_NEAR];
            total += W.step[TEAM_MEMBER];
            if (++iters > iter_cap)
                ok = false;
            mark(4);
        }

        // backward pass: the levels in reverse, down to the source's own
        if (ok) {
            int hi = band_start, lo = S.band_off[nlev - 1];
            for (int l = nlev - 1; l > 0 && ok; --l) {
                const int below = S.band_off[l - 1];
                PushCtx pc;
                pc.items = S.order + lo;
                pc.len = hi - lo;
                pc.worker = worker;
                pc.nworkers = nworkers;
                pc.marks = marks;
                pc.ebc = a.ebc;
                pc.emap = a.emap;
                push_level<PACKED, AG_SCOPE>(g, S, pc);
                hi = lo;
                lo = below;
                ok = team_barrier(W, y, par, band);
            }
            drounds += (unsigned long long)(nlev - 1);
            double *const bc = a.item_out ? a.item_out[idx] : a.bc_out;
            for (int v = gtid; ok && v < n; v += gn)
                if (S.d[v] != BC_INF) {
                    st_arcs += g.row[v + 1] - g.row[v];
                    if (v != s)
                        unsafeAtomicAdd(&bc[a.perm ? a.perm[v] : v], S.delta[v]);
                }
        }
        mark(3);
        if (lead) {
            if (!ok)
                atomicOr(&a.err[0], (unsigned long long)BC_ERRBIT_INTERNAL);
            atomicAdd(&a.stats->reached, (unsigned long long)band_start);
            atomicAdd(&a.stats->bands, (unsigned long long)nbands);
            atomicAdd(&a.stats->iterations, iters);
        }
        // a tripped bound is seen by every member; a failed barrier ends the team
        alive = W.failed == 0;
    }

    auto flush = [&](uint64_t x, unsigned long long *to) {
        for (int o = 32; o > 0; o >>= 1)
            x += __shfl_xor(x, o);
        if (lane_id() == 0 && x)
            atomicAdd(to, (unsigned long long)x);
    };
    flush(st_arcs, &a.stats->arcs);
    flush(st_dag, &a.stats->dag);
    flush(st_imp, &a.stats->improvements);
    if (threadIdx.x == 0 && W.failed)
        atomicOr(&a.err[0], (unsigned long long)BC_ERRBIT_INTERNAL);
    if (lead) {
        S.hdr[0] = gen;
        // after a failed barrier another member can be a round further on: the next
        // source clears the numbers
        S.hdr[1] = W.failed ? (1 << 30) + 1 : lvl;
        atomicAdd(&a.stats->sigma_rounds, srounds);
        atomicAdd(&a.stats->delta_rounds, drounds);
        for (int i = 0; i < 5; ++i)
            atomicAdd(&a.stats->ticks[i], ticks[i]);
    }
}

hipError_t launch_team(const TeamArgs &a, bool packed, hipStream_t st)
{
    const size_t words = sizeof(TeamCtl) * (size_t)a.teams / 4;
    const hipError_t e = launch_fill_u32((uint32_t *)a.ctl, words, 0u, st);
    if (e != hipSuccess)
        return e;
    const dim3 grid((unsigned)(a.teams * a.size)), block(TEAM_THREADS);
    const size_t lds = (size_t)a.bounds;
    const void *const k = packed ? (const void *)k_team<true> : (const void *)k_team<false>;
    if (lds > 48 * 1024)
        (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (packed)
        hipLaunchKernelGGL(k_team<true>, grid, block, lds, st, a);
    else
        hipLaunchKernelGGL(k_team<false>, grid, block, lds, st, a);
    return hipGetLastError();
}
