"""The hub kernel (single-vertex bitmap tiles of the 65535 top-ranked vertices; counts and batches of
at least 2^24 pairs and about 2^30 tail elements) against the oracle, at the edges of its rank range, its
16-byte chunks and its tiles, and just below the rules that lead to it."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tc():
    import paper_1804_06926_amd as tc
    return tc


def _dense(n, pairs, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    return rng.integers(0, n, size=(pairs, 2), dtype=np.int32)


PAIRS = 1 << 24   # the size rule


def _with_dense_core(n, pairs, core, seed, shift=0):
    """A complete graph on `core` vertices spread over [0, n) inside a random background; sum of C(d+, 2)
    is C(core, 3) and more, above 2^30 from core = 1900. `shift` drops that many pairs of the background."""
    rng = np.random.Generator(np.random.PCG64(seed))
    ids = rng.permutation(n)[:core].astype(np.int32)
    clique = ids[graphgen.complete(core)]
    e = np.concatenate([clique, rng.integers(0, n, size=(pairs - clique.shape[0] - shift, 2), dtype=np.int32)])
    return np.ascontiguousarray(e[rng.permutation(e.shape[0])]), n


GRAPHS = {
    # at the size rule and one pair below it
    "at_rule": lambda: _with_dense_core(1 << 21, PAIRS, 2100, 1),
    "below_rule": lambda: _with_dense_core(1 << 21, PAIRS, 2100, 1, shift=1),
    # few tail elements: the tiles stay with the bitmap kernel
    "below_tails": lambda: _with_dense_core(1 << 21, PAIRS, 600, 2),
    # vertices below, at and past the rank range; every vertex in it, tails of thousands of
    # elements, several tiles per vertex, rows of every alignment
    "n65534": lambda: _with_dense_core(65534, PAIRS, 2500, 3),
    "n65535": lambda: _with_dense_core(65535, PAIRS, 2500, 4),
    "n65536": lambda: _with_dense_core(65536, PAIRS + 3, 2500, 5),
    "n65537": lambda: _with_dense_core(65537, PAIRS, 2500, 6),
    "dense6000": lambda: (_dense(6000, PAIRS + 1, 7), 6000),
    "complete5800": lambda: (graphgen.complete(5800), 5800),
    # hubs joined to a pool and to vertices far below the rank range
    "spread": lambda: (np.ascontiguousarray(np.concatenate([graphgen.spread_hubs(),
                                                            _with_dense_core(1 << 21, PAIRS, 2000, 8)[0]])), 1 << 21),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_hub_counts(tc, name):
    import torch
    e, n = GRAPHS[name]()
    e = np.ascontiguousarray(e, dtype=np.int32)
    T = oracle.count_triangles(e, n)
    d = torch.from_numpy(e).cuda()
    for sel in (tc.SELECT_HEURISTIC, tc.FORCE_BITMAP):
        assert tc.count_triangles(d, n, select=sel) == T, sel


@pytest.mark.parametrize("graph", [True, False])
def test_hub_batch(tc, graph):
    """Per-graph sums through the hub kernel's per-vertex updates, replayed with other calls between."""
    import torch
    parts = [graphgen.rmat(14, 40, seed=1), graphgen.complete(2100), graphgen.chung_lu(200001, 14_000_007, seed=2),
             graphgen.star(9000), _dense(900, 200_001, 3)]
    nv = np.array([1 << 14, 2100, 200001, 9001, 900], dtype=np.int32)
    off = np.concatenate([[0], np.cumsum([p.shape[0] for p in parts])]).astype(np.int64)
    assert off[-1] >= PAIRS
    e = np.ascontiguousarray(np.concatenate(parts), dtype=np.int32)
    ref = np.array([oracle.count_triangles(np.ascontiguousarray(p, dtype=np.int32), int(n))
                    for p, n in zip(parts, nv)], dtype=np.uint64)
    d = torch.from_numpy(e).cuda()
    small = torch.from_numpy(graphgen.complete(50).astype(np.int32)).cuda()
    for _ in range(3):
        assert np.array_equal(tc.count_triangles_batch(d, off, nv, graph=graph), ref)
        assert tc.count_triangles(small, 50) == 19600
