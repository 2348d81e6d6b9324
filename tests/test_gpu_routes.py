"""The forms that calls take, as their statistics report them: each of the cases
that the other tests aim at does take the form it is there for."""
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


def batch(rnmod, net, specs, want):
    out, off, status = net.join_batch(specs)
    assert not status.any()
    for seg, w in zip(rnmod.split_batch(out, off), want):
        same(seg, w)
    return net.stats()["route"]


def test_degrees(rnmod, orc, rg):
    # 16 arcs a vertex are searched over quads, 17 over windows
    for degree, want in ((16, rnmod.RN_ROUTE_QUADS), (17, rnmod.RN_ROUTE_WINDOWS)):
        n = 300
        src = np.concatenate([np.arange(n - j) for j in range(1, degree + 1)])
        dst = np.concatenate([np.arange(j, n) for j in range(1, degree + 1)])
        g = rg.from_edges(n, src, dst, 1 + (src * 7 + dst) % 50, symmetric=False)
        net = rnmod.RoadNetwork.from_graph(g)
        R, S = rg.sample_disjoint(n, 20, 60, 1)
        same(rnmod.pairs_to_numpy(net.dist_join(R, S, 200)), orc.dist_join(g, R, S, 200).pairs)
        assert net.stats()["route"] & (rnmod.RN_ROUTE_QUADS | rnmod.RN_ROUTE_WINDOWS) == want


def test_short_form_and_guess(rnmod, orc, rg):
    g = rg.road_graph(150, 2)
    net = rnmod.RoadNetwork.from_graph(g)
    R, S = rg.sample_disjoint(g.V, 300, 300, 3)
    same(rnmod.pairs_to_numpy(net.dist_join(R, S, 900)), orc.dist_join(g, R, S, 900).pairs)
    assert net.stats()["route"] == rnmod.RN_ROUTE_QUADS | rnmod.RN_ROUTE_SHORT
    same(rnmod.pairs_to_numpy(net.kcp_join(R, S, 16)), orc.kcp_join(g, R, S, 16))
    assert net.stats()["route"] == rnmod.RN_ROUTE_QUADS | rnmod.RN_ROUTE_SHORT | rnmod.RN_ROUTE_GUESS
    # R among the first rows of the grid, S among the last
    Ra, Sa = np.arange(0, 1500, 7, dtype=np.int32), np.arange(g.V - 1500, g.V, 7, dtype=np.int32)
    same(rnmod.pairs_to_numpy(net.kcp_join(Ra, Sa, 9)), orc.kcp_join(g, Ra, Sa, 9))
    assert net.stats()["route"] & rnmod.RN_ROUTE_GUESS_MISSED
    # more searches, and more vertices, than the short form takes
    for nR, theta in ((5000, 900), (300, 4000)):
        R, S = rg.sample_disjoint(g.V, nR, 5000, 4)
        same(rnmod.pairs_to_numpy(net.dist_join(R, S, theta)), orc.dist_join(g, R, S, theta).pairs)
        assert not net.stats()["route"] & rnmod.RN_ROUTE_SHORT


def dense_patch(rg):
    """A path of long arcs, its first vertices joined by many short ones: balls
    and pair counts far above the estimate from the mean weight."""
    rng = np.random.default_rng(3)
    n, m = 8000, 2500
    path = np.arange(n - 1)
    cycles = [rng.permutation(m) for _ in range(3)]
    src = np.concatenate([path] + cycles)
    dst = np.concatenate([path + 1] + [np.roll(c, 1) for c in cycles])
    w = np.concatenate([rng.integers(400, 500, n - 1), rng.integers(1, 30, 3 * m)])
    return rg.from_edges(n, src, dst, w, symmetric=True), rng.permutation(m).astype(np.int32)


def test_short_form_hands_over(rnmod, orc, rg):
    g, ids = dense_patch(rg)
    net = rnmod.RoadNetwork.from_graph(g)
    left = rnmod.RN_ROUTE_SHORT | rnmod.RN_ROUTE_SHORT_LEFT
    # balls that outgrow the table; more records than the tail sorts; both
    for nR, nS, theta in ((30, 40, 300), (900, 900, 16), (120, 900, 60)):
        R, S = ids[:nR], ids[nR:nR + nS]
        same(rnmod.pairs_to_numpy(net.dist_join(R, S, theta)), orc.dist_join(g, R, S, theta).pairs)
        st = net.stats()
        assert st["route"] & left == left, (nR, nS, theta)
        assert (st["pairs"] > 4096) == (nR > 30) and (st["retried"] > 0) == (theta > 16), st


def flat_grid(rg):
    """Weights of 100 but for a few: most distances are multiples of 100."""
    g = rg.road_graph(120, 5)
    w = np.full(g.A, 100, dtype=np.uint32)
    w[:40] = 100 + np.arange(40)
    return rg.from_edges(g.V, np.repeat(np.arange(g.V), np.diff(g.row_ptr)), g.col, w, symmetric=False)


@pytest.mark.parametrize("kcp_first", [False, True])
def test_mixed_bins_too_full(rnmod, orc, rg, kcp_first):
    # several thousand pairs at one distance: beyond what the ranking takes
    g = flat_grid(rg)
    net = rnmod.RoadNetwork.from_graph(g)
    R, S = rg.sample_disjoint(g.V, 3000, 7000, 1)
    R2, S2 = rg.sample_disjoint(g.V, 400, 500, 2)
    specs, want = [{"R": R, "S": S, "theta": 300}], [orc.dist_join(g, R, S, 300).pairs]
    assert np.unique(want[0]["dist"], return_counts=True)[1].max() > 4096
    k = {"R": R2, "S": S2, "k": 2000}
    specs.insert(0 if kcp_first else 1, k)
    want.insert(0 if kcp_first else 1, orc.kcp_join(g, R2, S2, 2000))
    for _ in range(2):
        assert batch(rnmod, net, specs, want) & rnmod.RN_ROUTE_RESORTED


def test_theta_bins_too_full(rnmod, orc, rg):
    g = flat_grid(rg)
    net = rnmod.RoadNetwork.from_graph(g)
    R, S = rg.sample_disjoint(g.V, 3000, 7000, 1)
    same(rnmod.pairs_to_numpy(net.dist_join(R, S, 300)), orc.dist_join(g, R, S, 300).pairs)
    assert net.stats()["route"] & rnmod.RN_ROUTE_RESORTED


@pytest.mark.parametrize("beside", [0, 300])
def test_whole_graph_ring_full(rnmod, orc, rg, beside):
    # two random cycles through 100 000 vertices: tens of thousands pending at once
    n = 100000
    rng = np.random.default_rng(8)
    p, q = rng.permutation(n), rng.permutation(n)
    g = rg.from_edges(n, np.concatenate([p, q]), np.concatenate([np.roll(p, 1), np.roll(q, 1)]),
                      rng.integers(90, 111, size=2 * n), symmetric=True)
    net = rnmod.RoadNetwork.from_graph(g)
    R, S = np.array([0, n - 1, 500], dtype=np.int32), np.arange(1000, 3000, dtype=np.int32)
    specs, want = [{"R": R, "S": S, "hash_log2": rnmod.RN_TABLE_GLOBAL}], [orc.dist_join(g, R, S, 0xFFFFFFFE).pairs]
    if beside:
        R2 = np.arange(4000, 4000 + beside, dtype=np.int32)
        specs.append({"R": R2, "S": S, "theta": 600})
        want.append(orc.dist_join(g, R2, S, 600).pairs)
    batch(rnmod, net, specs, want)   # (allocates the tier's slots)
    assert batch(rnmod, net, specs, want) & rnmod.RN_ROUTE_DENSE_FULL
    # a road graph's searches stay within it
    g = rg.road_graph(130, 3)
    net = rnmod.RoadNetwork.from_graph(g)
    R, S = rg.sample_disjoint(g.V, 30, 200, 1)
    specs, want = [{"R": R, "S": S, "hash_log2": rnmod.RN_TABLE_GLOBAL}], [orc.dist_join(g, R, S, 0xFFFFFFFE).pairs]
    for _ in range(2):
        assert not batch(rnmod, net, specs, want) & rnmod.RN_ROUTE_DENSE_FULL
