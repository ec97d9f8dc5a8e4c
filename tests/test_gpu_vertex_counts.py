"""Per-vertex counts, clustering coefficients and edge support of graphs past the small-graph sizes,
at the edges of the LDS counters of the 2048 top ranks and of the 2048-element lists whose hits are
gathered in LDS, against the oracle and closed forms."""
import numpy as np
import pytest

import graphgen
import oracle
from oracle.measures import clustering

pytestmark = pytest.mark.gpu

PAIRS = (1 << 17) + 1   # one past the small-graph rule


@pytest.fixture(scope="module")
def tc():
    import paper_1804_06926_amd as tc
    return tc


def _random(n, pairs, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    return rng.integers(0, n, size=(pairs, 2), dtype=np.int32)


GRAPHS = {
    "n2047": lambda: (_random(2047, PAIRS, 1), 2047),
    "n2048": lambda: (_random(2048, PAIRS, 2), 2048),
    "n2049": lambda: (_random(2049, PAIRS, 3), 2049),
    # a hub over everything: its row-last count and t[w] pass through one counter
    "hub": lambda: (np.concatenate([graphgen.star(70000), _random(70001, 300000, 4)]).astype(np.int32), 70001),
    "rmat17": lambda: (graphgen.rmat(17, 16, seed=5), 1 << 17),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_vertex_counts_and_clustering(tc, name):
    import torch
    e, n = GRAPHS[name]()
    d = torch.from_numpy(np.ascontiguousarray(e)).cuda()
    r_coeff, r_T, r_W, r_tr, r_t = clustering(e, n)
    for sel in (tc.SELECT_HEURISTIC, tc.FORCE_BITMAP, tc.FORCE_BSEARCH):
        T, t = tc.count_triangles(d, n, per_vertex=True, select=sel)
        assert T == r_T
        np.testing.assert_array_equal(t.cpu().numpy().astype(np.uint64), r_t)
    coeff, T, W, tr = tc.clustering(d, n)
    assert (T, W, tr) == (r_T, r_W, r_tr)
    np.testing.assert_array_equal(coeff.cpu().numpy(), r_coeff)


@pytest.mark.parametrize("k", [2048, 2049, 2300])
def test_complete_graph_counts_and_support(tc, k):
    """Out-lists of up to k - 1 elements, on both sides of 2048: t[v] = C(k - 1, 2), support k - 2."""
    import torch
    d = torch.from_numpy(graphgen.complete(k).astype(np.int32)).cuda()
    T0 = k * (k - 1) * (k - 2) // 6
    for sel in (tc.SELECT_HEURISTIC, tc.FORCE_BSEARCH):
        T, t = tc.count_triangles(d, k, per_vertex=True, select=sel)
        assert T == T0 and bool((t == (k - 1) * (k - 2) // 2).all())
    pairs, sup, T = tc.edge_support(d, k)
    assert T == T0 and pairs.shape[0] == k * (k - 1) // 2 and bool((sup == k - 2).all())
    pairs, cnt, T = tc.edge_counts(d, k)
    assert T == T0 and int(cnt.to(torch.int64).sum()) == T0
