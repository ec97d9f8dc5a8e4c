"""Per-edge counts and support of the bitmap strategy where hits are rare, dense, and both in one round of long tails."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tc():
    import paper_1804_06926_amd as tc
    return tc


@pytest.mark.parametrize("dense", [0, 40, 300])
def test_rare_and_dense_hits(tc, dense):
    """A uniform graph of degree about 300 on 20,000 vertices (tails of 64 and more, about one hit in 70 items), with
    `dense` vertices joined to each other and to a tenth of the rest."""
    import torch
    n = 20_000
    rng = np.random.Generator(np.random.PCG64(dense))
    parts = [rng.integers(0, n, size=(3_000_000, 2))]
    if dense:
        a, b = np.triu_indices(dense, 1)
        parts.append(np.stack([a, b], 1))
        rest = rng.choice(np.arange(dense, n), size=n // 10, replace=False)
        parts.append(np.stack([np.repeat(np.arange(dense), rest.size), np.tile(rest, dense)], 1))
    e = np.concatenate(parts)
    e = rng.permutation(n)[e].astype(np.int32)
    e = np.ascontiguousarray(e[rng.permutation(len(e))])
    d = torch.from_numpy(e).cuda()
    T = oracle.count_triangles(e, n)
    want = {}
    for sel in (tc.FORCE_MERGE, tc.FORCE_BITMAP, tc.SELECT_HEURISTIC):
        pairs, counts, Tc = tc.edge_counts(d, n, select=sel)
        pairs2, support, Ts = tc.edge_support(d, n, select=sel)
        assert Tc == Ts == T
        assert int(counts.long().sum()) == T and int(support.long().sum()) == 3 * T
        for k, x in (("pairs", pairs), ("counts", counts), ("pairs2", pairs2), ("support", support)):
            assert torch.equal(want.setdefault(k, x.clone()), x), (sel, k)
