"""The hub group kernel (32 consecutive ones of the 16384 top-ranked vertices at a time, counts of at least 2^24 pairs and
about 2^30 tail elements): rows that hold one, several and all members of a group, groups cut by other strategies,
vertices of every row alignment, the smallest vertex count it takes."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tc():
    import paper_1804_06926_amd as tc
    return tc


PAIRS = 1 << 24


def _core(n, pairs, core, p, seed):
    """p times the pairs of `core` of n vertices, drawn at random (all of them for p = 1), in a random background."""
    rng = np.random.Generator(np.random.PCG64(seed))
    ids = rng.permutation(n)[:core].astype(np.int32)
    e = ids[graphgen.complete(core) if p == 1 else rng.integers(0, core, size=(int(p * core * core / 2), 2))]
    e = np.concatenate([e, rng.integers(0, n, size=(pairs - e.shape[0], 2), dtype=np.int32)])
    return np.ascontiguousarray(e[rng.permutation(e.shape[0])], dtype=np.int32)


CASES = {
    "one_member_in_twenty": lambda: (_core(1 << 20, PAIRS, 18000, 0.05, 1), 1 << 20),
    "half": lambda: (_core(300_001, PAIRS, 4000, 0.5, 2), 300_001),
    "all": lambda: (_core(65_535, PAIRS, 2300, 1.0, 3), 65_535),
    "odd": lambda: (_core(70_003, PAIRS + 5, 5500, 0.3, 4), 70_003),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_group_counts(tc, name):
    import torch
    e, n = CASES[name]()
    T = oracle.count_triangles(e, n)
    d = torch.from_numpy(e).cuda()
    for sel in (tc.SELECT_HEURISTIC, tc.FORCE_BITMAP, tc.FORCE_BSEARCH):
        assert tc.count_triangles(d, n, select=sel) == T, sel
    for chunk in (16, 128):   # other tile shapes: more and fewer single-vertex tiles
        tc.set_tile_shapes(np.full(256, chunk, dtype=np.uint16), None)
        try:
            assert tc.count_triangles(d, n) == T, chunk
        finally:
            tc.set_tile_shapes(None, None)
