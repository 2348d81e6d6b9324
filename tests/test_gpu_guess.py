"""k-closest-pairs queries whose searches start from a guessed bound, against the
oracle: where the guess holds, where R and S lie too far apart for it (the call
is run again without), in eager calls, batches, plans and the server."""
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


def apart(V, n, seed):
    """R among the first tenth of the ids (rows of the grid), S among the last."""
    rng = np.random.default_rng(seed)
    R = rng.choice(V // 10, size=n, replace=False).astype(np.int32)
    S = (V - 1 - rng.choice(V // 10, size=n, replace=False)).astype(np.int32)
    return R, S


def two_components(rg):
    a, b = rg.road_graph(60, 3), rg.road_graph(60, 4)
    src = np.concatenate([np.repeat(np.arange(a.V), np.diff(a.row_ptr)), a.V + np.repeat(np.arange(b.V), np.diff(b.row_ptr))])
    return rg.from_edges(a.V + b.V, src, np.concatenate([a.col, a.V + b.col]), np.concatenate([a.w, b.w]),
                         symmetric=False), a.V


@pytest.mark.parametrize("nR,nS", [(300, 300), (37, 2000), (2000, 37), (5, 5)])
def test_guess_holds_or_not(rnmod, orc, rg, nR, nS):
    g = rg.road_graph(150, 2)
    net = rnmod.RoadNetwork.from_graph(g)
    R, S = rg.sample_disjoint(g.V, nR, nS, nR)
    for k in (1, 3, 16, 100, 700, 2047, 2049):
        if k <= nR * nS:
            same(rnmod.pairs_to_numpy(net.kcp_join(R, S, k)), orc.kcp_join(g, R, S, k))
    R, S = apart(g.V, min(nR, nS, 300), 9)
    for k in (1, 9):
        same(rnmod.pairs_to_numpy(net.kcp_join(R, S, k)), orc.kcp_join(g, R, S, k))


def test_unreachable_pairs(rnmod, orc, rg):
    g, half = two_components(rg)
    net = rnmod.RoadNetwork.from_graph(g)
    rng = np.random.default_rng(5)
    R = rng.choice(half, size=200, replace=False).astype(np.int32)
    S = (half + rng.choice(g.V - half, size=200, replace=False)).astype(np.int32)
    assert len(rnmod.pairs_to_numpy(net.kcp_join(R, S, 10))) == 0


def test_batch_and_plan(rnmod, orc, rg):
    import torch
    g = rg.road_graph(150, 2)
    net = rnmod.RoadNetwork.from_graph(g)
    R1, S1 = rg.sample_disjoint(g.V, 400, 500, 1)
    R2, S2 = apart(g.V, 200, 2)
    specs = [{"R": R1, "S": S1, "k": 50}, {"R": R2, "S": S2, "k": 20}, {"R": R1, "S": S1, "theta": 500}]
    want = [orc.kcp_join(g, R1, S1, 50), orc.kcp_join(g, R2, S2, 20), orc.dist_join(g, R1, S1, 500).pairs]
    out, off, status = net.join_batch(specs)
    assert not status.any()
    for a, b in zip(rnmod.split_batch(out, off), want):
        same(a, b)
    # a plan whose sets move apart between replays, and back
    Rd, Sd = (torch.from_numpy(x.copy()).to("cuda") for x in (R1[:200], S1[:200]))
    queries, keep = net.make_queries([{"R": Rd, "S": Sd, "k": 30}])
    plan = net.plan(queries, cap=64)
    for R, S in ((R1[:200], S1[:200]), (R2, S2), (R1[200:400], S1[200:400])):
        Rd.copy_(torch.from_numpy(R.copy()))
        Sd.copy_(torch.from_numpy(S.copy()))
        for _ in range(2):
            got, off, _ = plan.run()
            same(rnmod.pairs_to_numpy(got), orc.kcp_join(g, R, S, 30))


def test_server(rnmod, orc, rg):
    g = rg.road_graph(150, 2)
    net = rnmod.RoadNetwork.from_graph(g)
    server = rnmod.Server(net)
    sets = [rg.sample_disjoint(g.V, 300, 200, 1), apart(g.V, 100, 3), rg.sample_disjoint(g.V, 80, 900, 4)]
    ids = [server.submit(R, S, k=25) for R, S in sets]
    for rid, (R, S) in zip(ids, sets):
        same(server.wait(rid)[0], orc.kcp_join(g, R, S, 25))
    server.close()


def test_one_missed_guess_among_others(rnmod, orc, rg):
    # R and S apart in an order of the ids that does not show it: the guess is
    # made and missed; the batch's and the server's other queries are not the worse
    g, perm = rg.shuffle_ids(rg.road_graph(150, 2), 5)[:2]
    net = rnmod.RoadNetwork.from_graph(g)
    R2, S2 = (perm[x].astype(np.int32) for x in apart(g.V, 200, 2))
    sets = [rg.sample_disjoint(g.V, 300, 400, i) for i in range(3)]
    specs = [{"R": R, "S": S, "k": 50 + i} for i, (R, S) in enumerate(sets)] + [{"R": R2, "S": S2, "k": 20}]
    want = [orc.kcp_join(g, sp["R"], sp["S"], sp["k"]) for sp in specs]
    for _ in range(2):
        out, off, status = net.join_batch(specs)
        assert not status.any()
        for a, b in zip(rnmod.split_batch(out, off), want):
            same(a, b)
        route = net.stats()["route"]
        assert route & rnmod.RN_ROUTE_GUESS and route & rnmod.RN_ROUTE_GUESS_MISSED
    q, keep = net.make_queries(specs)
    plan = net.plan(q, cap=sum(len(w) for w in want))
    for _ in range(3):
        got, off, _ = plan.run()
        for a, b in zip(rnmod.split_batch(got, off), want):
            same(a, b)
    plan.close()
    server = rnmod.Server(net, lanes=1)
    for _ in range(2):
        ids = [server.submit(sp["R"], sp["S"], k=sp["k"]) for sp in specs]
        for rid, w in zip(ids, want):
            same(server.wait(rid)[0], w)
    st = server.stats()
    assert st["reruns"] >= 2 and st["completed"] == 8, st
    server.close()
