"""One-query calls that take the one-block staging and tail, against the oracle:
sizes around a staging word, argument errors, more records than the tail sorts,
a search that outgrows its table, an output that does not fit."""
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


@pytest.mark.parametrize("side", [2, 5, 6, 9, 33, 64, 181, 182, 250])
def test_sizes(rnmod, orc, rg, side):
    g = rg.road_graph(side, side)
    net = rnmod.RoadNetwork.from_graph(g)
    for nR, nS in ((1, 1), (31, 33), (64, 64), (1500, 700), (4096, 4000)):
        if nR + nS > g.V:
            continue
        R, S = rg.sample_disjoint(g.V, nR, nS, side + nR)
        for theta in (0, 120, 700, 1500):
            same(rnmod.pairs_to_numpy(net.dist_join(R, S, theta)), orc.dist_join(g, R, S, theta).pairs)
        for k in (1, 7, 1000, 2048):
            if k <= nR * nS:
                same(rnmod.pairs_to_numpy(net.kcp_join(R, S, k)), orc.kcp_join(g, R, S, k))


def test_renumbered_and_reversed(rnmod, orc, rg):
    g = rg.shuffle_ids(rg.road_graph(120, 3), 4)[0]
    net = rnmod.RoadNetwork.from_graph(g)
    net.partition(alpha=0.5)
    d = rg.random_digraph(3000, 12000, 31, wmin=1, wmax=60, zero_frac=0.2)
    netd = rnmod.RoadNetwork.from_graph(d)
    for graph, n, theta in ((g, net, 900), (d, netd, 40)):
        for nR, nS in ((200, 300), (300, 40)):
            R, S = rg.sample_disjoint(graph.V, nR, nS, nS)
            same(rnmod.pairs_to_numpy(n.dist_join(R, S, theta)), orc.dist_join(graph, R, S, theta).pairs)
            same(rnmod.pairs_to_numpy(n.kcp_join(R, S, 40)), orc.kcp_join(graph, R, S, 40))


@pytest.mark.parametrize("bad", ["range", "negative", "dupR", "dupS", "overlap"])
def test_argument_errors(rnmod, orc, rg, bad):
    g = rg.road_graph(64, 0)
    net = rnmod.RoadNetwork.from_graph(g)
    R0, S0 = rg.sample_disjoint(g.V, 64, 64, 1)
    R, S = R0.copy(), S0.copy()
    if bad == "range":
        S[3] = g.V
    elif bad == "negative":
        R[3] = -1
    elif bad == "dupR":
        R[3] = R[4]
    elif bad == "dupS":
        S[3] = S[4]
    else:
        S[3] = R[4]
    for call in (lambda: net.dist_join(R, S, 900), lambda: net.kcp_join(R, S, 9)):
        with pytest.raises(rnmod.RnError) as ei:
            call()
        assert ei.value.status == rnmod.RN_ERR_ARG
    same(rnmod.pairs_to_numpy(net.dist_join(R0, S0, 900)), orc.dist_join(g, R0, S0, 900).pairs)


def test_more_records_or_vertices_than_expected(rnmod, orc, rg):
    # a dense patch in a sparse graph: balls and pair counts far above the
    # estimate from the mean weight, so the short form hands over; also as a plan
    rng = np.random.default_rng(3)
    n, m = 12000, 2500
    path = np.arange(n - 1)
    src = np.concatenate([path, rng.integers(0, m, 3 * m)])
    dst = np.concatenate([path + 1, rng.integers(0, m, 3 * m)])
    w = np.concatenate([rng.integers(400, 500, n - 1), rng.integers(1, 30, 3 * m)])
    keep = src != dst
    g = rg.from_edges(n, src[keep], dst[keep], w[keep], symmetric=True)
    net = rnmod.RoadNetwork.from_graph(g)
    ids = rng.permutation(m).astype(np.int32)
    for nR, nS in ((60, 60), (120, 900)):
        R, S = ids[:nR], ids[nR:nR + nS]
        for theta in (60, 300):
            want = orc.dist_join(g, R, S, theta).pairs
            same(rnmod.pairs_to_numpy(net.dist_join(R, S, theta)), want)
            queries, keepq = net.make_queries([{"R": R, "S": S, "theta": theta}])
            plan = net.plan(queries, cap=len(want) + 5)
            for _ in range(3):
                same(rnmod.pairs_to_numpy(plan.run()[0]), want)
        same(rnmod.pairs_to_numpy(net.kcp_join(R, S, 1500)), orc.kcp_join(g, R, S, 1500))
