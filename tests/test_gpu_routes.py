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
    # vertices of more than 16 arcs, or of more than half a further quad each on
    # average, are searched over windows; the others over quads
    def ring(n, reach):
        src = np.concatenate([np.arange(n) for _ in reach])
        dst = np.concatenate([(np.arange(n) + j) % n for j in reach])
        return rg.from_edges(n, src, dst, 1 + (src * 7 + dst) % 50, symmetric=True)

    def with_hubs(hubs, arcs):
        g = ring(900, (1, 2))        # 4 arcs a vertex
        src, dst = np.repeat(np.arange(900), np.diff(g.row_ptr)), g.col
        h = np.repeat(np.arange(hubs) * 2, arcs)
        to = (h + 5 + np.tile(np.arange(arcs), hubs)) % 900
        # (one way, so that the hubs' arcs add to few others' in the reversed graph)
        return rg.from_edges(900, np.concatenate([src, h]), np.concatenate([dst, to]),
                             np.concatenate([g.w, 1 + (h + to) % 50]), symmetric=False)

    q, w = rnmod.RN_ROUTE_QUADS, rnmod.RN_ROUTE_WINDOWS
    for g, want in ((ring(900, (1,)), q), (ring(900, (1, 2)), q), (ring(900, (1, 2, 3)), w),
                    (with_hubs(1, 12), q), (with_hubs(1, 13), w), (with_hubs(140, 4), q)):
        net = rnmod.RoadNetwork.from_graph(g)
        for nR, nS in ((20, 60), (60, 20)):
            R, S = rg.sample_disjoint(g.V, nR, nS, 1)
            same(rnmod.pairs_to_numpy(net.dist_join(R, S, 200)), orc.dist_join(g, R, S, 200).pairs)
            assert net.stats()["route"] & (q | w) == want, (g.A, want)


@pytest.mark.parametrize("parts", [2, 3, 8])
def test_chains_of_two_arcs(rnmod, orc, rg, parts):
    # a road graph whose edges are cut into parts: 2.5 to 2.1 arcs a vertex
    r = rg.road_graph(60, 3)
    src = np.repeat(np.arange(r.V), np.diff(r.row_ptr))
    m = src < r.col
    a, b, w = src[m], r.col[m], np.maximum(1, r.w[m] // parts)
    mids = r.V + np.arange(len(a) * (parts - 1)).reshape(len(a), parts - 1)
    chain = np.concatenate([a[:, None], mids, b[:, None]], axis=1)
    g = rg.from_edges(r.V + mids.size, chain[:, :-1].ravel(), chain[:, 1:].ravel(), np.repeat(w, parts), symmetric=True)
    net = rnmod.RoadNetwork.from_graph(g)
    for nR, nS in ((50, 300), (3000, 400), (5000, 5000)):
        R, S = rg.sample_disjoint(g.V, min(nR, g.V // 3), min(nS, g.V // 3), nR)
        for theta in (60, 300, 1200):
            same(rnmod.pairs_to_numpy(net.dist_join(R, S, theta)), orc.dist_join(g, R, S, theta).pairs)
            assert net.stats()["route"] & rnmod.RN_ROUTE_QUADS
        same(rnmod.pairs_to_numpy(net.kcp_join(R, S, 200)), orc.kcp_join(g, R, S, 200))
    for sp, want in (({"theta": 0xFFFFFFFE}, orc.dist_join(g, R[:20], S, 0xFFFFFFFE).pairs),
                     ({"k": 3000}, orc.kcp_join(g, R[:20], S, 3000))):
        for _ in range(2):
            out, off, status = net.join_batch([{"R": R[:20], "S": S, "hash_log2": rnmod.RN_TABLE_GLOBAL, **sp}])
            same(rnmod.pairs_to_numpy(out[:off[1]]), want)


def test_short_form_and_guess(rnmod, orc, rg):
    g = rg.road_graph(150, 2)
    net = rnmod.RoadNetwork.from_graph(g)
    R, S = rg.sample_disjoint(g.V, 300, 300, 3)
    same(rnmod.pairs_to_numpy(net.dist_join(R, S, 900)), orc.dist_join(g, R, S, 900).pairs)
    assert net.stats()["route"] == rnmod.RN_ROUTE_QUADS | rnmod.RN_ROUTE_SHORT
    same(rnmod.pairs_to_numpy(net.kcp_join(R, S, 40)), orc.kcp_join(g, R, S, 40))
    assert net.stats()["route"] == rnmod.RN_ROUTE_QUADS | rnmod.RN_ROUTE_SHORT | rnmod.RN_ROUTE_GUESS
    # R among the first rows of the grid, S among the last: no guess; the same in an
    # order of the ids that does not show it: a missed one
    Ra, Sa = np.arange(0, 1500, 7, dtype=np.int32), np.arange(g.V - 1500, g.V, 7, dtype=np.int32)
    same(rnmod.pairs_to_numpy(net.kcp_join(Ra, Sa, 9)), orc.kcp_join(g, Ra, Sa, 9))
    assert not net.stats()["route"] & (rnmod.RN_ROUTE_GUESS | rnmod.RN_ROUTE_GUESS_MISSED)
    h, perm = rg.shuffle_ids(g, 5)[:2]
    neth = rnmod.RoadNetwork.from_graph(h)
    Ra, Sa = perm[Ra].astype(np.int32), perm[Sa].astype(np.int32)
    same(rnmod.pairs_to_numpy(neth.kcp_join(Ra, Sa, 9)), orc.kcp_join(h, Ra, Sa, 9))
    assert neth.stats()["route"] & rnmod.RN_ROUTE_GUESS_MISSED
    # more searches, and more vertices, than the short form takes
    for nR, theta in ((5000, 900), (300, 4000)):
        R, S = rg.sample_disjoint(g.V, nR, 5000, 4)
        same(rnmod.pairs_to_numpy(net.dist_join(R, S, theta)), orc.dist_join(g, R, S, theta).pairs)
        assert not net.stats()["route"] & rnmod.RN_ROUTE_SHORT


@pytest.mark.parametrize("nR,nS,k", [(300, 300, 5), (1000, 1000, 100), (40, 20000, 30), (150, 150, 2), (6000, 6000, 1500)])
def test_sets_spread_alike_are_guessed(rnmod, orc, rg, nR, nS, k):
    # one block of ids after another, up to blocks of 2 048; also beside other queries
    g = rg.road_graph(330, 2)
    net = rnmod.RoadNetwork.from_graph(g)
    made = 0
    for seed in range(6):
        R, S = rg.sample_disjoint(g.V, nR, nS, seed)
        want = orc.kcp_join(g, R, S, k)
        same(rnmod.pairs_to_numpy(net.kcp_join(R, S, k)), want)
        made += (net.stats()["route"] & rnmod.RN_ROUTE_GUESS) != 0
        specs = [{"R": R[:50], "S": S[:50], "theta": 300}, {"R": R, "S": S, "k": k}]
        batch(rnmod, net, specs, [orc.dist_join(g, R[:50], S[:50], 300).pairs, want])
        made += (net.stats()["route"] & rnmod.RN_ROUTE_GUESS) != 0
    assert made == 12


def dense_patch(rg, n, seed=3):
    """A road graph, n vertices of it joined by short arcs: balls and pair counts
    far above the estimate from the mean weight.  (From id 700 on: between two of
    the 32 places where loading looks how dense the graph is, when n <= 1000.)"""
    rng = np.random.default_rng(seed)
    r = rg.road_graph(200, 5)
    cycles = [700 + rng.permutation(n) for _ in range(3)]
    src = np.concatenate([np.repeat(np.arange(r.V), np.diff(r.row_ptr))] + cycles + [np.roll(c, 1) for c in cycles])
    dst = np.concatenate([r.col] + [np.roll(c, 1) for c in cycles] + cycles)
    w = rng.integers(1, 6, 3 * n)
    g = rg.from_edges(r.V, src, dst, np.concatenate([r.w, w, w]), symmetric=False)
    return g, 700 + rng.permutation(n).astype(np.int32)


def test_short_form_hands_over(rnmod, orc, rg):
    g, ids = dense_patch(rg, 1000)
    net = rnmod.RoadNetwork.from_graph(g)
    left = rnmod.RN_ROUTE_QUADS | rnmod.RN_ROUTE_SHORT | rnmod.RN_ROUTE_SHORT_LEFT
    # balls that outgrow the table; more records than the tail sorts; both
    for nR, nS, theta in ((30, 40, 60), (450, 450, 5), (120, 850, 60)):
        R, S = ids[:nR], ids[nR:nR + nS]
        want = orc.dist_join(g, R, S, theta).pairs
        for _ in range(2):
            same(rnmod.pairs_to_numpy(net.dist_join(R, S, theta)), want)
            st = net.stats()
            assert st["route"] & ~(rnmod.RN_ROUTE_RESORTED | rnmod.RN_ROUTE_BINS) == left, (nR, nS, theta)
            assert (st["pairs"] > 4096) == (nR > 30) and (st["retried"] > 0) == (theta > 5), st
        # (from the first run of a plan on, it is captured in the general form)
        q, keep = net.make_queries([{"R": R, "S": S, "theta": theta}])
        plan = net.plan(q, cap=len(want))
        for _ in range(3):
            same(rnmod.pairs_to_numpy(plan.run()[0]), want)
        plan.close()
    # k closest pairs whose balls outgrow the table
    R, S = ids[:300], ids[300:700]
    same(rnmod.pairs_to_numpy(net.kcp_join(R, S, 900)), orc.kcp_join(g, R, S, 900))
    assert net.stats()["route"] & left == left


def test_plan_hands_over_in_a_replay(rnmod, orc, rg):
    # sets that lie in the sparse part when the plan is made, then in the dense one
    import torch
    g, ids = dense_patch(rg, 1000)
    net = rnmod.RoadNetwork.from_graph(g)
    far = 20000 + np.arange(500, dtype=np.int32)
    Rd, Sd = torch.from_numpy(far[:100].copy()).cuda(), torch.from_numpy(far[100:].copy()).cuda()
    q, keep = net.make_queries([{"R": Rd, "S": Sd, "theta": 60}])
    plan = net.plan(q, cap=100000)
    for R, S in ((far[:100], far[100:]), (ids[:100], ids[100:500]), (far[:100], far[100:])):
        Rd.copy_(torch.from_numpy(R.copy()))
        Sd.copy_(torch.from_numpy(S.copy()))
        torch.cuda.synchronize()
        for _ in range(2):
            same(rnmod.pairs_to_numpy(plan.run()[0]), orc.dist_join(g, R, S, 60).pairs)
    plan.close()


def test_tables_hold_the_densest_part(rnmod, orc, rg):
    # a fifth of a road graph with arcs a quarter as long, and queries in it: the
    # tables are large enough, in the short form and beyond it
    r = rg.road_graph(300, 0)
    src = np.repeat(np.arange(r.V), np.diff(r.row_ptr))
    lo, hi = int(.4 * r.V), int(.6 * r.V)
    w = np.where((src >= lo) & (src < hi) & (r.col >= lo) & (r.col < hi), np.maximum(1, r.w // 4), r.w)
    g = rg.from_edges(r.V, src, r.col, w, symmetric=False)
    net = rnmod.RoadNetwork.from_graph(g)
    ids = lo + np.random.default_rng(4).permutation(hi - lo).astype(np.int32)
    for nR, theta in ((30, 500), (1000, 250), (5000, 500), (6000, 250)):
        R, S = ids[:nR], ids[nR:2 * nR]
        same(rnmod.pairs_to_numpy(net.dist_join(R, S, theta)), orc.dist_join(g, R, S, theta).pairs)
        assert net.stats()["retried"] == 0, (nR, theta)
    # (a guess of 30 vertices a ball on average)
    R, S = ids[:500], ids[500:1500]
    same(rnmod.pairs_to_numpy(net.kcp_join(R, S, 100)), orc.kcp_join(g, R, S, 100))
    st = net.stats()
    assert st["route"] & rnmod.RN_ROUTE_GUESS and st["retried"] == 0, st


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
    R, S = rg.sample_disjoint(g.V, 3000, 5000, 1)
    R2, S2 = rg.sample_disjoint(g.V, 400, 500, 2)
    specs, want = [{"R": R, "S": S, "theta": 300}], [orc.dist_join(g, R, S, 300).pairs]
    assert np.unique(want[0]["dist"], return_counts=True)[1].max() > 4096
    k = {"R": R2, "S": S2, "k": 2000}
    specs.insert(0 if kcp_first else 1, k)
    want.insert(0 if kcp_first else 1, orc.kcp_join(g, R2, S2, 2000))
    for _ in range(2):
        assert batch(rnmod, net, specs, want) & rnmod.RN_ROUTE_RESORTED


@pytest.mark.parametrize("nR,nS,theta,bins", [(300, 500, 2000, True), (3000, 3000, 300, True), (3000, 3000, 700, True),
                                              (5000, 5000, 700, False), (5000, 5000, 2000, False),
                                              (200, 300, 0xFFFFFFFE, False)])
@pytest.mark.parametrize("nq", [1, 6])
def test_long_bins_are_not_made(rnmod, orc, rg, nR, nS, theta, bins, nq):
    # a theta-join beside closest-pairs queries: binned where few pairs share one
    g = rg.road_graph(120, 3)
    net = rnmod.RoadNetwork.from_graph(g)
    R, S = rg.sample_disjoint(g.V, nR, nS, 1)
    specs, want = [{"R": R, "S": S, "theta": theta}], [orc.dist_join(g, R, S, theta).pairs]
    for i in range(nq):
        R2, S2 = rg.sample_disjoint(g.V, 400, 500, 2 + i)
        specs.insert(i % 2, {"R": R2, "S": S2, "k": 1500})
        want.insert(i % 2, orc.kcp_join(g, R2, S2, 1500))
    for _ in range(2):
        route = batch(rnmod, net, specs, want)
        assert bool(route & rnmod.RN_ROUTE_BINS) == bins and not route & rnmod.RN_ROUTE_RESORTED


@pytest.mark.parametrize("nR,nS,k,bins", [(1500, 1500, 3000, True), (4500, 9000, 30000, False), (400, 500, 100000, True)])
def test_long_bins_of_closest_pairs_are_not_made(rnmod, orc, rg, nR, nS, k, bins):
    g = rg.road_graph(120, 3)
    net = rnmod.RoadNetwork.from_graph(g)
    R, S = rg.sample_disjoint(g.V, nR, nS, 1)
    for _ in range(2):
        same(rnmod.pairs_to_numpy(net.kcp_join(R, S, k)), orc.kcp_join(g, R, S, k))
        assert bool(net.stats()["route"] & rnmod.RN_ROUTE_BINS) == bins


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
