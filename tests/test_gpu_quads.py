"""Searches over arc quads (graphs of at most 16 arcs per vertex) against the
oracle, where they can go wrong: vertices with one to four quads, the first
degree beyond them (searched over arc windows), every table size, graphs of
different sizes in one launch, small tables whose searches share a stage."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rnmod():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1607_07696_amd import rn
    rn.load_library()
    return rn


def same(got, want):
    assert got.shape == want.shape and np.array_equal(got, want)


def clique_chain(rg, degree, n, seed, directed=False):
    """n vertices whose out-degrees run up to `degree` (arcs to the next ids)."""
    rng = np.random.default_rng(seed)
    src, dst = [], []
    for x in range(n):
        for j in range(1, degree // (1 if directed else 2) + 1):
            if x + j < n:
                src.append(x)
                dst.append(x + j)
    w = rng.integers(1, 90, size=len(src))
    return rg.from_edges(n, np.array(src), np.array(dst), w, symmetric=not directed)


@pytest.mark.parametrize("directed", [False, True])
@pytest.mark.parametrize("degree", [4, 5, 6, 8, 10, 12, 14, 16, 17, 18])
def test_degrees(rnmod, orc, rg, degree, directed):
    g = clique_chain(rg, degree, 700, degree, directed)
    net = rnmod.RoadNetwork.from_graph(g)
    for nR, nS in ((40, 300), (300, 40)):      # the second searches the reversed arcs
        R, S = rg.sample_disjoint(g.V, nR, nS, degree + nR)
        for theta in (0, 50, 400, 3000):
            same(rnmod.pairs_to_numpy(net.dist_join(R, S, theta)), orc.dist_join(g, R, S, theta).pairs)
        same(rnmod.pairs_to_numpy(net.kcp_join(R, S, 777)), orc.kcp_join(g, R, S, 777))


@pytest.mark.parametrize("hb", range(8, 15))
def test_graphs_of_different_sizes_in_one_launch(rnmod, orc, rg, hb):
    graphs = [rg.road_graph(90, 1), rg.road_graph(9, 2), clique_chain(rg, 16, 400, 3), rg.road_graph(40, 4),
              rg.road_graph(5, 5)]
    net = rnmod.RoadNetwork.from_graphs(graphs)
    specs = []
    for i, g in enumerate(graphs):
        R, S = rg.sample_disjoint(g.V, min(200, g.V // 2), min(300, g.V // 3), i)
        for theta in (300, 1100):
            specs.append({"R": R, "S": S, "theta": theta, "graph": i, "hash_log2": hb})
    out, off, status = net.join_batch(specs)
    assert not status.any()
    for sp, seg in zip(specs, rnmod.split_batch(out, off)):
        same(seg, orc.dist_join(graphs[sp["graph"]], sp["R"], sp["S"], sp["theta"]).pairs)


@pytest.mark.parametrize("theta", [1, 250, 500, 700, 900, 1200, 1600, 2300, 2900])
def test_tables_chosen_by_radius(rnmod, orc, rg, theta):
    # dense and sparse targets: a stage of 64 pairs fills within one search, over
    # several, or holds them to the end; many more sources than blocks
    g = rg.road_graph(160, 7)
    net = rnmod.RoadNetwork.from_graph(g)
    for nR, nS in ((12000, 13000) if theta <= 900 else (9000, 900), (9000, 40), (63, 65)):
        R, S = rg.sample_disjoint(g.V, nR, nS, theta)
        same(rnmod.pairs_to_numpy(net.dist_join(R, S, theta)), orc.dist_join(g, R, S, theta).pairs)


def test_global_tier_over_quads(rnmod, orc, rg):
    # whole-graph searches in the global tier: pairs found by S's list, by the
    # vertices reached, and of a graph whose pending sets outgrow the search's ring of
    # 16 384 entries (it goes on to the general global tier)
    g = rg.road_graph(130, 3)
    net = rnmod.RoadNetwork.from_graph(g)
    for nR, nS in ((30, 200), (20, 9000), (65, 300)):   # (the last: more searches than it takes)
        R, S = rg.sample_disjoint(g.V, nR, nS, nS)
        for sp, want in (({"theta": 0xFFFFFFFE}, orc.dist_join(g, R, S, 0xFFFFFFFE).pairs),
                         ({"theta": 5000}, orc.dist_join(g, R, S, 5000).pairs), ({"k": 3000}, orc.kcp_join(g, R, S, 3000))):
            out, off, status = net.join_batch([{"R": R, "S": S, "hash_log2": rnmod.RN_TABLE_GLOBAL, **sp}])
            assert not status.any()
            same(rnmod.pairs_to_numpy(out[:off[1]]), want)
    # two random cycles through 100 000 vertices: tens of thousands pending at once
    n = 100000
    rng = np.random.default_rng(8)
    p, q = rng.permutation(n), rng.permutation(n)
    t = rg.from_edges(n, np.concatenate([p, q]), np.concatenate([np.roll(p, 1), np.roll(q, 1)]),
                      rng.integers(90, 111, size=2 * n), symmetric=True)
    net = rnmod.RoadNetwork.from_graph(t)
    net.set_profiling(times=True, work=True)
    R = np.array([0, n - 1, 500], dtype=np.int32)
    S = np.arange(1000, 3000, dtype=np.int32)
    out, off, status = net.join_batch([{"R": R, "S": S, "hash_log2": rnmod.RN_TABLE_GLOBAL},
                                       {"R": R, "S": S, "k": 500, "hash_log2": rnmod.RN_TABLE_GLOBAL}])
    segs = rnmod.split_batch(out, off)
    ref = orc.dist_join(t, R, S, 0xFFFFFFFE)
    same(segs[0], ref.pairs)
    same(segs[1], orc.kcp_join(t, R, S, 500))
