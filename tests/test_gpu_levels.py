"""The batched form's flat expansion, candidate batches and level passes at the
edges of their tiles: queue lengths and degrees around the wavefront width and
the workgroup's waves, vertices without out-arcs between others, hubs, and ties
in every position of the recorded predecessor lists."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1701_05975_amd import bc, graphgen as gg

pytestmark = pytest.mark.gpu


def layered(width: int, degrees, seed: int):
    """Source 0 -> `width` queued vertices of the given degrees (cycled; 0
    included) -> a pool of heads that lead back into one vertex; small weights,
    so heads are offered equal, better and worse distances."""
    rng = np.random.default_rng(seed)
    deg = np.resize(np.asarray(degrees), width)
    pool = max(int(deg.max()), 70) + 7
    n = 1 + width + pool + 1
    src = [np.zeros(width, np.int64)]
    dst = [1 + np.arange(width)]
    for i, d in enumerate(deg):
        src.append(np.full(d, 1 + i))
        dst.append(1 + width + rng.choice(pool, size=d, replace=False))
    src.append(1 + width + np.arange(pool))
    dst.append(np.full(pool, n - 1))
    src, dst = np.concatenate(src), np.concatenate(dst)
    return gg.csr_from_arcs(n, src, dst, rng.integers(1, 4, size=src.shape[0]), directed=True)


@pytest.mark.parametrize("width", [1, 15, 16, 17, 63, 64, 65, 1023, 1025, 2049])
@pytest.mark.parametrize("degrees", [[1], [0, 3], [63, 64, 65], [0, 0, 127, 1, 129], [2, 700, 5]],
                         ids=str)
def test_layers(width, degrees):
    if width > 1100 and max(degrees) > 200:
        pytest.skip("covered by the smaller widths")
    g = layered(width, degrees, seed=width + len(degrees))
    srcs = np.concatenate([np.zeros(3, np.int64), np.arange(0, g.n, max(1, g.n // 40))])
    want = oracle.oracle_bc(g, srcs)
    G = bc.Graph(g)
    for opts in (dict(), dict(wg_threads=1024, delta=1), dict(delta=1, far_buckets=1),
                 dict(lane_max_deg=1, wg_min_deg=64), dict(accumulate=2), dict(dep_mode=2),
                 dict(keep=1)):
        H = bc.Graph(g, keep_order=True) if opts.pop("keep", 0) else G
        got, st = H.bc(srcs, **opts)
        # sums of at most a few thousand non-negative terms: 1e-16 relative each
        assert np.all(got[want == 0] == 0)
        nz = want != 0
        assert nz.sum() == 0 or np.max(np.abs(got[nz] - want[nz]) / want[nz]) <= 1e-11, opts
        d, sg, _ = H.source_state(0, **opts)
        od, osg, _, _ = oracle.oracle_source_state(g, 0)
        od = np.where(od == np.iinfo(np.int64).max, 2**31 - 1, od)
        assert np.array_equal(d, od) and np.array_equal(sg, osg), opts
    G.close()


def narrow_layers(width: int, seed: int):
    """A tree of at most 8 arcs a vertex whose leaves, all queued in one step, are
    `width`; each leaf has 0 to 8 arcs to a pool, with small weights."""
    rng = np.random.default_rng(seed)
    sizes = [width]
    while sizes[-1] > 1:
        sizes.append((sizes[-1] + 7) // 8)
    src, dst, w, first = [], [], [], 0
    for up, down in zip(sizes[:0:-1], sizes[-2::-1]):
        src.append(first + np.arange(down) * up // down)
        dst.append(first + up + np.arange(down))
        w.append(np.ones(down, np.int64))
        first += up
    deg = rng.integers(0, 9, width)
    pool = width + 9
    src.append(np.repeat(first + np.arange(width), deg))
    dst.append(first + width + np.concatenate(
        [rng.choice(pool, d, replace=False) for d in deg]).astype(np.int64))
    w.append(rng.integers(1, 4, int(deg.sum())))
    src.append(first + width + np.arange(pool))
    dst.append(np.full(pool, first + width + pool))
    w.append(rng.integers(1, 4, pool))
    return gg.csr_from_arcs(first + width + pool + 1, np.concatenate(src), np.concatenate(dst),
                            np.concatenate(w), directed=True)


@pytest.mark.parametrize("threads", [256, 512, 1024])
@pytest.mark.parametrize("off", [-1, 0, 1])
def test_narrow_queues(threads, off):
    """Queues at the length up to which groups of four lanes expand them."""
    g = narrow_layers(threads // 4 + off, seed=threads + off)
    assert np.diff(g.row_ptr).max() <= 8
    srcs = np.concatenate([np.zeros(3, np.int64), np.arange(0, g.n, max(1, g.n // 40))])
    want = oracle.oracle_bc(g, srcs)
    G = bc.Graph(g)
    for opts in (dict(), dict(delta=1), dict(delta=1, far_buckets=1), dict(accumulate=2)):
        got, _ = G.bc(srcs, wg_threads=threads, **opts)
        assert np.all(got[want == 0] == 0)
        nz = want != 0
        assert np.max(np.abs(got[nz] - want[nz]) / want[nz]) <= 1e-11, opts
    G.close()


@pytest.mark.parametrize("n, hub", [(300, 64), (640, 0), (1024, 0)])
@pytest.mark.parametrize("threads", [256, 1024])
def test_hubs_that_improve_each_other(n, hub, threads):
    """Complete graphs, every vertex a hub: their distances fall while their own
    lists are expanded, in one wide band or in many."""
    rng = np.random.default_rng(n)
    a, b = np.triu_indices(n, 1)
    w = rng.integers(1, 1001, a.shape[0])
    g = gg.csr_from_arcs(n, np.concatenate([a, b]), np.concatenate([b, a]),
                         np.concatenate([w, w]), directed=False, m=a.shape[0])
    srcs = np.array([0, n // 2, n - 1, 0], np.int32)
    want = oracle.oracle_bc(g, srcs)
    od, osg, _, _ = oracle.oracle_source_state(g, 1)
    G = bc.Graph(g)
    for opts in (dict(), dict(delta=1 << 20), dict(delta=3, far_buckets=1),
                 dict(far_buckets=2, lds_bits=16), dict(delta=1 << 20, lds_bits=8),
                 dict(delta=16, lds_bits=8, far_buckets=2)):
        got, st = G.bc(srcs, wg_threads=threads, wg_min_deg=hub, **opts)
        assert st["lds_vertices"] > 0
        assert np.all(got[want == 0] == 0)
        nz = want != 0
        # sums of at most a few thousand non-negative terms: 1e-16 relative each
        assert np.max(np.abs(got[nz] - want[nz]) / want[nz]) <= 1e-11, opts
        d, sg, _ = G.source_state(1, wg_threads=threads, wg_min_deg=hub, **opts)
        assert np.array_equal(d, od) and np.array_equal(sg, osg), opts
    G.close()


def lattice(side: int, hub_arcs: int):
    """A grid whose middle vertex has `hub_arcs` more arcs."""
    i = np.arange(side * side).reshape(side, side)
    c = int(i[side // 2, side // 2])
    far = np.setdiff1d(np.arange(c - side // 3, c + side // 3), [c - 1, c, c + 1])[:hub_arcs]
    u = np.concatenate([i[:, :-1].ravel(), i[:-1].ravel(), np.full(far.shape[0], c)])
    v = np.concatenate([i[:, 1:].ravel(), i[1:].ravel(), far])
    w = np.random.default_rng(side).integers(1, 256, u.shape[0])
    return gg.undirected_from_edges(side * side, u, v, w)


@pytest.mark.parametrize("side, hub_arcs", [(60, 6), (300, 6), (300, 60)])
def test_one_wide_vertex_changes_no_plan(side, hub_arcs):
    """A grid is handled as one whether or not a few of its vertices have more than 8
    arcs: the same threads, no team, and nearly the same band width."""
    torch = pytest.importorskip("torch")
    plain, wide = lattice(side, 0), lattice(side, hub_arcs)
    P, W = bc.Graph(plain), bc.Graph(wide)
    rp, col, w = (torch.from_numpy(a).cuda() for a in (wide.row_ptr, wide.col, wide.w))
    torch.cuda.synchronize()
    D = bc.Graph.from_device(wide, rp, col, w, stream=torch.cuda.current_stream().cuda_stream)
    for k in (1, 300, 600):
        s = np.resize(np.array([0, side, plain.n - 1], np.int32), k)
        (_, a), (got, b), (_, d) = (G.bc(s) for G in (P, W, D))
        for f in ("wg_threads", "lds_vertices"):
            assert a[f] == b[f] == d[f], (f, k)
        assert b["lds_vertices"] > 0 and b["delta"] == d["delta"]
        assert abs(a["delta"] - b["delta"]) <= 0.05 * a["delta"], k
        want = sum(np.count_nonzero(s == v) * oracle.oracle_bc(wide, np.array([v]))
                   for v in np.unique(s))
        nz = want != 0
        assert np.max(np.abs(got[nz] - want[nz]) / want[nz]) <= 1e-11
    for G in (P, W, D):
        G.close()


@pytest.mark.parametrize("n", [300, 700])
def test_bands_of_dense_graphs(n):
    """The bands of a dense graph are not much wider than its paths are long: eight
    maximum weights over the degree at most, five times that for a team."""
    a, b = np.triu_indices(n, 1)
    g = gg.undirected_from_edges(n, a, b, np.random.default_rng(n).integers(1, 1001, a.shape[0]))
    G = bc.Graph(g)
    for k, team in ((n, 1), (64, 1), (1, 5)):
        s = np.arange(k, dtype=np.int32)
        got, st = G.bc(s)
        assert 1 <= st["delta"] <= team * 8 * 1000 / (n - 1), (k, st["delta"])
        want = oracle.oracle_bc(g, s)
        nz = want != 0
        assert np.max(np.abs(got[nz] - want[nz]) / want[nz]) <= 1e-11
    G.close()


@pytest.mark.parametrize("n, threads", [(8192, 512), (8193, 1024)])
def test_threads_of_small_random_graphs(n, threads):
    """Random graphs of up to 65536 arcs with more sources than compute units."""
    g = gg.er_graph(n, 4 * n, 1, 100, seed=n)
    assert g.nnz == 8 * n
    G = bc.Graph(g)
    s = np.resize(np.array([0, 5, n - 1], np.int32), 300)
    got, st = G.bc(s)
    assert st["wg_threads"] == threads
    assert G.bc(s[:256])[1]["wg_threads"] == 1024
    want = 100 * oracle.oracle_bc(g, s[:3])
    nz = want != 0
    assert np.max(np.abs(got[nz] - want[nz]) / want[nz]) <= 1e-11
    G.close()
