"""The wave kernel (vertices of fewer than 1024 in-edges, counts and batches of at least 2^24 pairs): middle lists whose
ranks all fall on one slot of its table, below and above what its table of whole ranks takes at once; its
vertex limit; mixed degrees against the oracle."""
import math

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

SLOTS, TAGS = 2048, 0x7FFF


@pytest.fixture(scope="module")
def tc():
    import paper_1804_06926_amd as tc
    return tc


def _classes(k, classes=SLOTS):
    """`classes` complete graphs on k vertices, ids SLOTS apart within one. All degrees are equal, so ranks are in id
    order and a middle list's ranks differ by multiples of SLOTS."""
    base = graphgen.complete(k).astype(np.int64) * SLOTS
    e = (base[None] + np.arange(classes)[:, None, None]).reshape(-1, 2)
    return e.astype(np.int32)


@pytest.mark.parametrize("k", [129, 130, 194, 256])
@pytest.mark.parametrize("extra", [0, 1])
def test_one_slot(tc, k, extra):
    """C(k, 3) triangles per class; with `extra` the ids start past isolated vertices at an odd place."""
    import torch
    e = _classes(k)
    n = k * SLOTS
    if e.shape[0] < 1 << 24:   # repeat pairs of one class: their degrees rise, its ranks stay in order
        e = np.concatenate([e, e[:(1 << 24) - e.shape[0]]])
    if extra:
        e = e + np.int32(12345)
        n += 12345 + 7
    d = torch.from_numpy(np.ascontiguousarray(e)).cuda()
    T = SLOTS * math.comb(k, 3)
    for sel in (tc.SELECT_HEURISTIC, tc.FORCE_BITMAP):
        assert tc.count_triangles(d, n, select=sel) == T, sel


@pytest.mark.parametrize("n", [TAGS * SLOTS - 1, TAGS * SLOTS, TAGS * SLOTS + 1])
def test_vertex_limit(tc, n):
    import torch
    e = _classes(131) + np.int32(n - 131 * SLOTS)
    assert e.shape[0] >= 1 << 24
    d = torch.from_numpy(np.ascontiguousarray(e)).cuda()
    assert tc.count_triangles(d, n) == SLOTS * math.comb(131, 3)


@pytest.mark.parametrize("name", ["chung_lu", "rmat", "many"])
def test_against_the_oracle(tc, name):
    import torch
    if name == "chung_lu":
        n, e = 400_003, graphgen.chung_lu(400_003, (1 << 24) + 9, seed=3)
    elif name == "rmat":
        n, e = 1 << 19, graphgen.rmat(19, 33, seed=4)
    else:   # 300 to 1100 in-edges and more, below the hub ranks, in a dense graph
        n = 120_001
        e = np.random.Generator(np.random.PCG64(5)).integers(0, n, size=(60_000_000, 2), dtype=np.int32)
    e = np.ascontiguousarray(e, dtype=np.int32)
    assert e.shape[0] >= 1 << 24
    T = oracle.count_triangles(e, n)
    d = torch.from_numpy(e).cuda()
    for sel in (tc.SELECT_HEURISTIC, tc.FORCE_BITMAP):
        assert tc.count_triangles(d, n, select=sel) == T, sel


def test_batch(tc):
    import torch
    parts = [_classes(132), graphgen.complete(300), graphgen.chung_lu(50_001, 900_001, seed=6)]
    nv = np.array([132 * SLOTS, 300, 50_001], dtype=np.int32)
    off = np.concatenate([[0], np.cumsum([p.shape[0] for p in parts])]).astype(np.int64)
    e = np.ascontiguousarray(np.concatenate(parts), dtype=np.int32)
    d = torch.from_numpy(e).cuda()
    got = np.asarray(tc.count_triangles_batch(d, off, nv))
    want = [SLOTS * math.comb(132, 3), math.comb(300, 3), oracle.count_triangles(np.ascontiguousarray(parts[2], dtype=np.int32), 50_001)]
    assert got.tolist() == want
