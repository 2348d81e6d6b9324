"""A batch whose queries take every table size there is, theta-joins and guessed
k closest pairs side by side with whole-graph searches: as many first-tier
launches as a call can need."""
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


def run(rnmod, net, specs, want):
    for _ in range(2):
        out, off, status = net.join_batch(specs)
        assert not status.any()
        for seg, w in zip(rnmod.split_batch(out, off), want):
            same(seg, w)
    # 15 first-tier launches, a re-run tier, the global tier
    assert net.stats()["relax_launches"] >= 17


def test_every_table_size_in_one_call(rnmod, orc, rg):
    # (sizes set by the caller: what prepare would choose by itself needs
    # thousands of searches a size to keep them apart)
    g = rg.road_graph(150, 2)
    net = rnmod.RoadNetwork.from_graph(g)
    specs, want = [], []
    for hb in list(range(8, 15)) + [rnmod.RN_TABLE_GLOBAL]:
        R, S = rg.sample_disjoint(g.V, 120 + hb, 150, hb)
        for sp in ({"theta": 700}, {"k": 40}):
            specs.append({"R": R, "S": S, "hash_log2": hb, **sp})
            want.append(orc.kcp_join(g, R, S, 40) if "k" in sp else orc.dist_join(g, R, S, 700).pairs)
    run(rnmod, net, specs, want)


def test_sizes_chosen_by_the_library(rnmod, orc, rg):
    # theta-joins of seven ball sizes and k closest pairs of seven, thousands of
    # searches each, and one query of whole-graph searches
    g = rg.road_graph(700, 2)
    net = rnmod.RoadNetwork.from_graph(g)
    rng = np.random.default_rng(5)
    specs, want = [], []

    def add(nR, nS, **kw):
        R, S = rg.sample_disjoint(g.V, nR, nS, int(rng.integers(1 << 30)))
        specs.append({"R": R, "S": S, **kw})
        want.append(orc.kcp_join(g, R, S, kw["k"]) if "k" in kw else orc.dist_join(g, R, S, kw["theta"]).pairs)

    for theta in (600, 1050, 1500, 2100, 3400, 5000, 7300):      # 2^8 .. 2^14
        add(*((8300, 8300) if theta < 2200 else (300, 40)), theta=theta)
    for ball in (60, 200, 400, 800, 1600, 3200, 6500):           # 2^8 .. 2^14
        # a guess aims at 1.5 k + 8 pairs: (1.5 k + 8) V / (nR nS) vertices a ball
        nR, nS = (8300, 8300) if ball <= 800 else (300, 400)
        add(nR, nS, k=int((ball * nR * nS / g.V - 8) / 1.5))
    add(20, 30, k=500)
    run(rnmod, net, specs, want)
