"""The batched form with several workgroups per source: short source lists on
graphs large enough for it, against the oracle and against one workgroup per
source (wg_threads set)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1701_05975_amd import bc, graphgen as gg

pytestmark = pytest.mark.gpu


def close(got, want, tol):
    assert np.all(got[want == 0] == 0)
    nz = want != 0
    assert nz.sum() == 0 or np.max(np.abs(got[nz] - want[nz]) / want[nz]) <= tol


def tie_graph(n: int, seed: int):
    """Weights 1-2, parallel arcs and a hub of 3000 arcs: many predecessors, and
    the hub step of the expansion."""
    rng = np.random.default_rng(seed)
    src = np.concatenate([rng.integers(0, n, 12 * n), np.zeros(3000, np.int64),
                          rng.integers(0, n, 3000)])
    dst = np.concatenate([rng.integers(0, n, 12 * n), rng.integers(1, n, 3000),
                          np.zeros(3000, np.int64)])
    return gg.csr_from_arcs(n, src, dst, rng.integers(1, 3, src.shape[0]), directed=True)


GRAPHS = {
    # 360k: teams of 16 up to 8 sources; 1.3M: teams of 8 at 16 sources; 4.2M:
    # teams of 4 at 64 sources
    "er40k": (lambda: gg.er_graph(40_000, 160_000, 1, 100, seed=61), (1, 8)),
    "ties": (lambda: tie_graph(30_000, 62), (1, 3)),
    "ba110k": (lambda: gg.ba_graph(110_000, 5, 1, 1000, seed=63), (2, 16)),
    "rmat18": (lambda: gg.rmat_graph(18, 16 << 18, .57, .19, .19, 1, 255, seed=64), (5, 64)),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_team_matches_oracle(name):
    build, ks = GRAPHS[name]
    g = build()
    G = bc.Graph(g)
    for k in ks:
        s = gg.sample_sources(g, k, seed=k)
        s[-1] = s[0]  # a repeated source counts twice
        got, st = G.bc(s)
        assert st["wg_threads"] == 1024 and st["batch"] == k and st["lds_vertices"] == 0, st
        close(got, oracle.oracle_bc(g, s), 1e-11)
        one, st1 = G.bc(s, wg_threads=1024)
        assert st1["lds_vertices"] > 0
        for f in ("reached", "arcs_out_reached", "dag_arcs"):
            assert st[f] == st1[f], f
        close(got, one, 1e-11)
    for v in (int(s[0]), int(s[1]) if len(s) > 1 else 0):
        d, sg, dl = G.source_state(v)
        od, osg, odl, _ = oracle.oracle_source_state(g, v)
        assert np.array_equal(d, np.where(od == np.iinfo(np.int64).max, 2**31 - 1, od))
        assert np.array_equal(sg, osg)
        close(dl, odl, 1e-12)
    G.close()


@pytest.mark.parametrize("hubs", [1, 63, 64, 65, 4095, 4097])
def test_team_hub_list(hubs):
    """A queue with as many hubs as a group of 64, one more and one less, and
    as the list holds (4096)."""
    rng = np.random.default_rng(hubs)
    n, deg, tails = 300_000, 1100, np.arange(1, hubs + 1)
    src = np.concatenate([np.zeros(hubs, np.int64), np.repeat(tails, deg)])
    dst = np.concatenate([tails, rng.integers(5000, 8000, hubs * deg)])
    w = np.concatenate([np.ones(hubs, np.int64), rng.integers(1, 4, hubs * deg)])
    g = gg.csr_from_arcs(n, src, dst, w, directed=True)
    G = bc.Graph(g)
    s = np.array([0, 1], np.int32)
    got, st = G.bc(s)
    assert st["lds_vertices"] == 0, st
    close(got, oracle.oracle_bc(g, s), 1e-11)
    G.close()


@pytest.mark.parametrize("n, m, whi", [(40_000, 160_000, 50_000), (200_000, 400_000, 10_000),
                                        (200_000, 400_000, 1)])
def test_team_distance_bounds(n, m, whi):
    """Bounds with a unit above one and of one, more vertices than have a bound
    (n = 200,000), arcs that are not packed (n = 40,000)."""
    g = gg.er_graph(n, m, 1, whi, seed=67)
    G = bc.Graph(g)
    for delta in (0, max(whi // 50, 1), 8 * whi):
        s = gg.sample_sources(g, 3, seed=3)
        got, st = G.bc(s, delta=delta)
        assert st["lds_vertices"] == 0, st
        close(got, oracle.oracle_bc(g, s), 1e-11)
    G.close()


@pytest.mark.parametrize("n, m, k", [(200_000, 2_000_000, 80), (200_000, 2_000_000, 128),
                                     (80_000, 800_000, 32), (60_000, 600_000, 25)])
def test_small_teams(n, m, k):
    """Teams of two and three on the largest graphs, of every compute unit on the
    middle ones."""
    g = gg.er_graph(n, m, 1, 100, seed=68)
    G = bc.Graph(g)
    four = gg.sample_sources(g, 4, seed=4)
    s = np.resize(four, k)
    want = sum(np.count_nonzero(s == v) * oracle.oracle_bc(g, np.array([v])) for v in four)
    got, st = G.bc(s)
    assert st["lds_vertices"] == 0, st
    close(got, want, 1e-11)
    G.close()


def test_team_edges_and_errors():
    torch = pytest.importorskip("torch")
    g = gg.er_graph(40_000, 160_000, 1, 5, seed=65)
    G = bc.Graph(g, edges=True)
    s = gg.sample_sources(g, 6, seed=1)
    got, ebc = G.edge_bc(s)
    want, ewant = oracle.oracle_bc_edges(g, s)
    close(got, want, 1e-11)
    close(ebc, ewant, 1e-11)
    out = torch.empty(g.n, dtype=torch.float64, device="cuda")
    bad = torch.tensor([3, g.n, 5], dtype=torch.int32, device="cuda")
    with pytest.raises(bc.BCError) as ei:
        bc.bc_compute_device(G.handle, bad.data_ptr(), 3, out.data_ptr())
    assert ei.value.status == bc.BC_E_INVAL
    close(G.bc(s)[0], want, 1e-11)  # still usable
    G.close()


def test_team_reports_count_overflow():
    chain = gg.diamond_chain(64)  # 2^64 paths end to end
    rest = gg.er_graph(40_000, 160_000, 1, 100, seed=66)
    tail = np.repeat(np.arange(chain.n), np.diff(chain.row_ptr))
    rtail = np.repeat(np.arange(rest.n), np.diff(rest.row_ptr))
    g = gg.csr_from_arcs(chain.n + rest.n, np.concatenate([tail, rtail + chain.n]),
                         np.concatenate([chain.col, rest.col + chain.n]),
                         np.concatenate([chain.w, rest.w]), directed=False,
                         m=(chain.nnz + rest.nnz) // 2)
    G = bc.Graph(g)
    with pytest.raises(bc.BCError) as ei:
        G.bc(np.array([chain.n + 1, 0], np.int32))
    assert ei.value.status == bc.BC_E_SIGMA_OVERFLOW and "index 1" in ei.value.msg
    s = np.array([1, chain.n + 5], np.int32)
    close(G.bc(s)[0], oracle.oracle_bc(g, s), 1e-11)
    G.close()
