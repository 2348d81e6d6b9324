"""rn_autotune keeps the table that a query takes by itself where none of the other
settings is faster."""
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


def test_automatic_settings_are_among_those_tried(rnmod, orc, rg):
    # searches of a few dozen vertices: no other table or bucket width can be
    # faster by a tenth than the automatic one
    g = rg.road_graph(300, 3)
    net = rnmod.RoadNetwork.from_graph(g)
    specs, want = [], []
    for i in range(8):
        R, S = rg.sample_disjoint(g.V, 2000, 2500, i)
        specs.append({"R": R, "S": S, **({"k": 300} if i % 2 else {"theta": 600})})
        want.append(orc.kcp_join(g, R, S, 300) if i % 2 else orc.dist_join(g, R, S, 600).pairs)
    q, keep = net.make_queries(specs)
    net.autotune(q, sample=256)
    # (2^8 slots: for theta-joins not among the fixed sizes tried)
    assert sum(x.hash_log2 == 8 for x in q) >= 6, [(x.delta, x.hash_log2) for x in q]
    out, off, status = net.join_batch(q)
    assert not status.any()
    for seg, w in zip(rnmod.split_batch(out, off), want):
        assert seg.shape == w.shape and np.array_equal(seg, w)

