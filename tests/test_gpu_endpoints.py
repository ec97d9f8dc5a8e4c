"""The degree count's partition of the pairs: vertex counts about the widths of its 16-bit ids and of its single
pass, pair counts about its tiles, loops, and pairs with an invalid id."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tc():
    import paper_1804_06926_amd as tc
    return tc


SIZES = [(4097, 1), (4097, 16384), (65537, 1023), (65537, 2_097_151), (1 << 20, 1024), ((1 << 20) + 1, 2_097_153),
         (1 << 24, 1025), ((1 << 24) + 1, 2049), (1 << 24, 16_777_217), (1 << 25, 4097)]


@pytest.mark.parametrize("order", ["random", "sorted"])
@pytest.mark.parametrize("n,pairs", SIZES + [((1 << 24) + 1, 4_194_305)])
def test_ranks(tc, n, pairs, order):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n + pairs)
    e = torch.randint(0, n, (pairs, 2), generator=g, device="cuda", dtype=torch.int32)
    r = torch.rand(pairs, generator=g, device="cuda")
    e[r < 0.2, 0] = n - 1       # the vertex that takes the loops' endpoints until they are subtracted
    e[r > 0.9, 1] = e[r > 0.9, 0]
    if order == "sorted":   # whole waves of one digit
        e = e[torch.argsort(e[:, 0])].contiguous()
        e[:, 1] = torch.minimum(e[:, 0] + 1 + e[:, 1] % 97, torch.tensor(n - 1, device="cuda", dtype=torch.int32))
    deg = torch.bincount(e[e[:, 0] != e[:, 1]].flatten().long(), minlength=n)
    want = torch.empty(n, dtype=torch.int64, device="cuda")
    want[torch.argsort(deg, stable=True)] = torch.arange(n, device="cuda")
    rank, off, col = tc.build_csr(e, n)
    assert torch.equal(rank.long(), want)


@pytest.mark.parametrize("n", [20_000, (1 << 20) + 1, 1 << 24])
@pytest.mark.parametrize("bad", [-1, None, 2**31 - 1])
def test_invalid_ids(tc, n, bad):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    e = torch.randint(0, n, (300_001, 2), generator=g, device="cuda", dtype=torch.int32)
    good = e.clone()
    e[200_000, 1] = n if bad is None else bad
    with pytest.raises(tc.TCError) as err:
        tc.count_triangles(e, n)
    assert err.value.status == 2   # TC_ERR_VERTEX_RANGE
    tc.count_triangles(good, n)
