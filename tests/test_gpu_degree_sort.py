"""Sorts around the size from which their later passes look back (2^25 keys), and the degree order of graphs
whose buckets of endpoints are split over several blocks or counted in parts (24- and 25-bit ids)."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tc():
    import paper_1804_06926_amd as tc
    return tc


@pytest.mark.parametrize("count,lo,hi", [((1 << 25) - 1, 3, 25), (1 << 25, 0, 16), (1 << 25, 7, 29),
                                         ((1 << 25) + 8191, 0, 32), ((1 << 25) + 8193, 40, 56)])
def test_sort_around_the_look_back_size(tc, count, lo, hi):
    """Stable on the given bits; skewed digits, so that tiles hold long runs of one digit."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(count + lo)
    r = torch.rand(count, generator=g, device="cuda", dtype=torch.float64)
    field = (r ** 6 * float(1 << (hi - lo))).long().clamp_(max=(1 << (hi - lo)) - 1)
    keys = (field << lo) | (torch.arange(count, device="cuda") & ((1 << lo) - 1))
    if hi < 50:   # the position above the sorted bits shows the order of equal keys
        keys |= torch.arange(count, device="cuda") >> lo << hi if lo else torch.arange(count, device="cuda") << hi
    want = keys[torch.sort(field, stable=True).indices]
    got = tc.radix_sort_u64(keys.clone(), lo, hi)
    assert bool((got == want).all())


def _skewed(n, pairs, hubs, seed):
    """A third of all endpoints on a few hubs, the rest uniform; triangles through the hubs."""
    rng = np.random.Generator(np.random.PCG64(seed))
    e = rng.integers(0, n, size=(pairs, 2), dtype=np.int64)
    ids = rng.integers(0, n, size=hubs)
    third = rng.random(pairs) < 2.0 / 3.0
    e[third, 0] = ids[rng.integers(0, hubs, size=int(third.sum()))]
    near = rng.random(pairs) < 0.3
    e[near, 1] = ids[0] // 2 + rng.integers(0, 500, size=int(near.sum()))
    return np.ascontiguousarray(e, dtype=np.int32)


@pytest.mark.parametrize("n,pairs,hubs", [(5000, 150_000, 1), (300_001, 1_000_003, 2), ((1 << 20) - 3, 3_000_001, 1),
                                          ((1 << 24) - 5, 900_001, 1), ((1 << 24) + 3, 1_200_001, 3),
                                          ((1 << 25) - 1, 700_003, 1), ((1 << 25) + 9, 600_001, 2)])
def test_degree_order_with_hub_buckets(tc, n, pairs, hubs):
    """The exported rank is the position in (input degree, id) order."""
    import torch
    e = _skewed(n, pairs, hubs, n + pairs)
    d = torch.from_numpy(e).cuda()
    keep = d[:, 0] != d[:, 1]
    deg = torch.bincount(d[keep].flatten().long(), minlength=n)
    order = torch.argsort(deg, stable=True)
    want = torch.empty(n, dtype=torch.int32, device="cuda")
    want[order] = torch.arange(n, dtype=torch.int32, device="cuda")
    rank, off, col = tc.build_csr(d, n)
    assert bool((rank == want).all())
    assert tc.count_triangles(d, n, select=tc.FORCE_BSEARCH) == oracle.count_triangles(e, n)
