"""Block searches over quads leave their ring clear: rows read entries past the
last, which have to name quads of the next search's graph, and that may be far
smaller and lie at the end of the handle's."""
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


@pytest.mark.parametrize("hb,theta,side", [(12, 4000, 400), (13, 5500, 400), (14, 7500, 400)])
def test_large_searches_then_small_ones(rnmod, orc, rg, hb, theta, side):
    # the large graph's searches append thousands of entries, so that every place
    # of the ring has held one; then each block goes on with the small graphs'
    big, small = rg.road_graph(side, 1), [rg.road_graph(s, s) for s in (30, 12, 5)]
    graphs = [big] + small
    net = rnmod.RoadNetwork.from_graphs(graphs)
    specs, want = [], []
    for i, g in enumerate(graphs):
        R, S = rg.sample_disjoint(g.V, 3000 if i == 0 else g.V // 2, 200 if i == 0 else g.V // 3, i)
        for th in (theta, theta // 3):
            specs.append({"R": R, "S": S, "theta": th, "graph": i, "hash_log2": hb, "forward": True})
            want.append(orc.dist_join(g, R, S, th).pairs)
    for _ in range(2):
        out, off, status = net.join_batch(specs)
        assert not status.any()
        for seg, w in zip(rnmod.split_batch(out, off), want):
            assert seg.shape == w.shape and np.array_equal(seg, w)
