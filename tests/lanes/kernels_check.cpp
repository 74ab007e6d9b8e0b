// The batched kernels, run on the CPU (hip/hip_runtime.h beside this file) with
// guard words behind every array of a state slab.  Prints OK, or what is wrong.
//   kernels_check batched n degree wmax delta wg_deg seed group
//   kernels_check team n degree wmax delta wg_deg seed teams members clock_step looks
#include <algorithm>
#include <cmath>
#include <queue>
#include <string>

#include <hip/hip_runtime.h>

thread_local uint32_t lds_dist[40 * 1024], seen_bounds[40 * 1024];

#define BC_FOR_EACH_BATCHED(X) \
    X(true, 256, true, 32, false) X(true, 256, true, 16, true) X(true, 256, true, 8, false)
#include "kernels.hip"
#include "team.hip"

namespace {

struct Graph { // undirected, packed arcs, weights to wmax
    int n;
    std::vector<uint32_t> row, arc;
    uint32_t wshift, wmask;
    int maxdeg = 0;
    uint32_t head(uint32_t e) const { return arc[e] >> wshift; }
    uint32_t weight(uint32_t e) const { return (arc[e] & wmask) + 1; }
};

// Every vertex joined to `degree` of the next ones, and by a tail of single arcs.
Graph make_graph(int n, int degree, int wmax, unsigned seed)
{
    std::mt19937 rng(seed);
    std::vector<std::vector<std::pair<int, int>>> out(n);
    auto join = [&](int u, int v) {
        const int w = 1 + (int)(rng() % (unsigned)wmax);
        out[u].push_back({v, w});
        out[v].push_back({u, w});
    };
    const int core = n - n / 8;
    for (int u = 0; u < core; ++u)
        for (int j = 1; j <= degree / 2; ++j)
            if ((u + j) % core != u)
                join(u, (u + j) % core);
    for (int u = core; u < n; ++u)
        join(u, u - 1);
    Graph g;
    g.n = n;
    g.wshift = 0;
    while ((1 << g.wshift) < wmax)
        ++g.wshift;
    g.wmask = (1u << g.wshift) - 1;
    g.row.push_back(0);
    for (auto &o : out) {
        for (auto &a : o)
            g.arc.push_back((uint32_t)a.first << g.wshift | (uint32_t)(a.second - 1));
        g.row.push_back((uint32_t)g.arc.size());
        g.maxdeg = std::max(g.maxdeg, (int)o.size());
    }
    return g;
}

std::vector<double> brandes(const Graph &g, const std::vector<int32_t> &sources)
{
    std::vector<double> bc(g.n, 0.0);
    for (int s : sources) {
        std::vector<uint64_t> d(g.n, UINT64_MAX), sigma(g.n, 0);
        std::vector<double> delta(g.n, 0.0);
        std::priority_queue<std::pair<uint64_t, int>, std::vector<std::pair<uint64_t, int>>,
                            std::greater<>> q;
        d[s] = 0;
        sigma[s] = 1;
        q.push({0, s});
        std::vector<int> order;
        std::vector<char> done(g.n, 0);
        while (!q.empty()) {
            const int v = q.top().second;
            q.pop();
            if (done[v])
                continue;
            done[v] = 1;
            order.push_back(v);
            for (uint32_t e = g.row[v]; e < g.row[v + 1]; ++e) {
                const int u = (int)g.head(e);
                const uint64_t nd = d[v] + g.weight(e);
                if (nd < d[u]) {
                    d[u] = nd;
                    sigma[u] = 0;
                    q.push({nd, u});
                }
                if (nd == d[u])
                    sigma[u] += sigma[v];
            }
        }
        for (size_t i = order.size(); i-- > 0;) {
            const int v = order[i];
            for (uint32_t e = g.row[v]; e < g.row[v + 1]; ++e)
                if (d[g.head(e)] == d[v] + g.weight(e))
                    delta[v] += (double)sigma[v] / (double)sigma[g.head(e)] *
                                (1.0 + delta[g.head(e)]);
            if (v != s)
                bc[v] += delta[v];
        }
    }
    return bc;
}

constexpr uint32_t GUARD = 0xdeadbeefu;

struct Run {
    BatchArgs a;
    std::vector<char> slabs;
    std::vector<double> bc;
    std::vector<int32_t> sources;
    DevStats stats{};
    unsigned long long next = 0, err[2] = {0, ~0ull >> 1};
    std::vector<std::pair<size_t, const char *>> guards; // where one starts, behind what
    size_t guard_bytes;
    int nslabs;

    Run(const Graph &g, const std::vector<int32_t> &src, int slabs_wanted, int delta)
        : sources(src), nslabs(slabs_wanted)
    {
        const size_t n = (size_t)g.n;
        guard_bytes = 64 * n;
        SlabLayout L;
        size_t at = 0;
        auto take = [&](size_t bytes, const char *what, bool guard = true) {
            const size_t here = at;
            at += (bytes + 7) / 8 * 8;
            if (guard) {
                guards.push_back({here + bytes, what});
                at += guard_bytes;
            }
            return here;
        };
        L.d = take(4 * n, "d");
        L.rec = take(VREC_BYTES * n, "records");
        L.bcp = take(8 * n, "partial sums");
        L.order = take(4 * n, "order");
        L.qa = take(4 * n, "queue a");
        L.qb = take(4 * n, "queue b");
        L.fa = take(4 * n, "far a", false);
        L.fb = take(4 * n, "far b", false);
        L.bx = take(8 * n, "bucket pool");
        L.oa = take(4 * n, "outer a");
        L.ob = take(4 * n, "outer b");
        L.band_off = take(4 * (n + 2), "levels");
        L.hdr = take(64, "header");
        L.preds = take(4 * g.arc.size(), "predecessors");
        L.stride = (at + 255) / 256 * 256;
        slabs.resize(L.stride * (size_t)nslabs);
        bc.assign(n, 0.0);
        a.g = DevGraph{g.row.data(), g.arc.data(), nullptr, g.row.data(), g.arc.data(), nullptr,
                       g.n, g.n, g.wshift, g.wmask};
        a.slab_base = slabs.data();
        a.L = L;
        a.sources = sources.data();
        a.k = (long long)sources.size();
        a.next_src = &next;
        a.bc_out = bc.data();
        a.item_out = nullptr;
        a.item_err = nullptr;
        a.iperm = a.perm = nullptr;
        a.push = 1;
        a.vw = 0;
        a.node_parallel = 0;
        a.ebc = nullptr;
        a.emap = nullptr;
        a.delta = (uint32_t)delta;
        a.lane_max = 32;
        a.stats = &stats;
        a.err = err;
        reset();
    }

    void reset()
    {
        uint32_t *const w = (uint32_t *)slabs.data();
        std::fill(w, w + slabs.size() / 4, 0u);
        for (int i = 0; i < nslabs; ++i)
            for (auto &x : guards) {
                uint32_t *const p = (uint32_t *)(slabs.data() + i * a.L.stride + x.first);
                std::fill(p, p + guard_bytes / 4, GUARD);
            }
        std::fill(bc.begin(), bc.end(), 0.0);
        next = 0;
        err[0] = 0;
    }

    std::string check(const Graph &g)
    {
        for (int i = 0; i < nslabs; ++i)
            for (auto &x : guards) {
                const uint32_t *const p =
                    (const uint32_t *)(slabs.data() + i * a.L.stride + x.first);
                size_t past = 0;
                for (size_t j = 0; j < guard_bytes / 4; ++j)
                    past = p[j] != GUARD ? j + 1 : past;
                if (past)
                    return std::string("written past ") + x.second + ": " +
                           std::to_string(past) + " words";
            }
        if (err[0])
            return "error bits " + std::to_string(err[0]);
        const std::vector<double> want = brandes(g, sources);
        for (int v = 0; v < g.n; ++v)
            if (!(std::fabs(bc[v] - want[v]) <= 1e-11 * want[v]))
                return "centrality of " + std::to_string(v) + ": " + std::to_string(bc[v]) +
                       ", not " + std::to_string(want[v]);
        return "";
    }
};

// group: lanes per vertex in the expansion (0: arcs laid out flat, -1: flat, but
// short queues in small groups).
int batched(int n, int degree, int wmax, int delta, int wg_deg, unsigned seed, int group)
{
    const Graph g = make_graph(n, degree, wmax, seed);
    Run r(g, {0, n / 2, n - 1}, 1, delta);
    for (int lb : {32, 16, 8}) {
        r.reset();
        r.a.H = n - n / 16;
        r.a.lds_bits = lb;
        r.a.buckets = lb == 16;
        r.a.nbk = std::min((wmax + delta - 1) / delta + 2, BC_BUCKETS_MAX);
        r.a.bcap = 4 * n / r.a.nbk;
        r.a.wg_deg = (uint32_t)wg_deg;
        r.a.hubs = g.maxdeg > wg_deg;
        r.a.narrow = group < 0;
        r.a.vw = group < 0 ? 0 : group;
        if (launch_batched(r.a, true, 256, true, 1, nullptr) != hipSuccess)
            return printf("no such kernel\n"), 1;
        const std::string bad = r.check(g);
        if (!bad.empty())
            return printf("%d-bit distances: %s\n", lb, bad.c_str()), 1;
    }
    return 0;
}

// clock_step: ticks of the device clock between two reads of it, once the teams
// have formed.  looks: at a barrier, before a member takes it for failed (0: the
// library's own); a team whose barrier failed has to say so.
int team(int n, int degree, int wmax, int delta, int wg_deg, unsigned seed, int teams, int members,
         int clock_step, int looks)
{
    const Graph g = make_graph(n, degree, wmax, seed);
    Run r(g, {0, n / 2, n - 1}, teams, delta);
    r.a.H = 0;
    r.a.lds_bits = 32;
    r.a.wg_deg = (uint32_t)wg_deg;
    r.a.hubs = g.maxdeg > wg_deg;
    r.a.narrow = 0;
    std::vector<TeamCtl> ctl(teams);
    TeamArgs t;
    t.b = r.a;
    t.ctl = ctl.data();
    t.teams = teams;
    t.size = members;
    t.bounds = (n / 2 + 15) / 16 * 16;
    t.bshift = 0;
    while (((SEEN_WIN - SEEN_REBASE) << t.bshift) < (uint32_t)(wmax + delta))
        ++t.bshift;
    t.looks = looks > 0 ? (unsigned)looks : TEAM_WAIT_LOOKS;
    lanes::clock_step() = [&]() -> long long {
        for (auto &c : ctl)
            if (lanes::load(&c.members) == 0)
                return 1;
        return clock_step;
    };
    if (launch_team(t, true, nullptr) != hipSuccess)
        return printf("launch\n"), 1;
    for (auto &c : ctl)
        if (looks > 0 && c.failed) {
            if (r.err[0] != BC_ERRBIT_INTERNAL)
                return printf("a barrier failed without an error\n"), 1;
            printf("a barrier failed, ");
            return 0;
        }
    const std::string bad = r.check(g);
    return bad.empty() ? 0 : (printf("%s\n", bad.c_str()), 1);
}

} // namespace

int main(int argc, char **argv)
{
    int v[10] = {};
    if (argc != 9 && argc != 12)
        return 2;
    for (int i = 2; i < argc; ++i)
        v[i - 2] = atoi(argv[i]);
    lanes::seed() = (unsigned)v[5];
    int r = 2;
    if (!strcmp(argv[1], "batched"))
        r = batched(v[0], v[1], v[2], v[3], v[4], (unsigned)v[5], v[6]);
    else if (!strcmp(argv[1], "team"))
        r = team(v[0], v[1], v[2], v[3], v[4], (unsigned)v[5], v[6], v[7], v[8], v[9]);
    if (r == 0)
        printf("OK\n");
    return r;
}
