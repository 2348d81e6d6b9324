"""The first lightest of parallel arcs is found for rows compared pair by pair (up
to 16 arcs) as for longer, sorted ones: closest pairs of direct arcs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree", [2, 15, 16, 17, 40])
def test_rows_of_parallel_arcs(orc, rg, degree):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1607_07696_amd import rn
    rng = np.random.default_rng(degree)
    n = 300
    rows = np.arange(n + 1, dtype=np.int32) * degree
    # each vertex has arcs to few others, many of them equal
    col = ((np.arange(n)[:, None] + 1 + rng.integers(0, 3, (n, degree))) % n).astype(np.int32).ravel()
    w = rng.integers(90, 94, n * degree).astype(np.uint32)
    g = rg.Graph(rows, col, w)
    net = rn.RoadNetwork.from_graph(g)
    for nR, nS in ((100, 150), (150, 100)):
        R, S = rg.sample_disjoint(n, nR, nS, degree)
        for k in (3, 40):
            got, want = rn.pairs_to_numpy(net.kcp_join(R, S, k)), orc.kcp_join(g, R, S, k)
            assert got.shape == want.shape and np.array_equal(got, want)
