"""The degree order where many vertices have a degree past the sorted range (65535 and more): repeated pairs on few
vertices, about one comparison block of 256 and several, with equal degrees among them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tc():
    import paper_1804_06926_amd as tc
    return tc


@pytest.mark.parametrize("hubs,others", [(255, 0), (256, 1), (257, 1000), (700, 100_000), (1030, 513)])
def test_rank_among_many_hubs(tc, hubs, others):
    """Hub i is joined to hub i + 1 (in a ring) 32738 + r_i times, r_i in [0, 60), so that degrees repeat and some may fall
    short of the bound, and the other vertices to the hubs once each; ids are permuted."""
    import torch
    n = hubs + others
    rng = np.random.Generator(np.random.PCG64(hubs))
    times = torch.from_numpy(32738 + rng.integers(0, 60, size=hubs)).cuda()
    a = torch.repeat_interleave(torch.arange(hubs, device="cuda"), times)
    d = torch.stack([a, (a + 1) % hubs], 1)
    if others:
        o = torch.arange(hubs, n, device="cuda")
        d = torch.cat([d, torch.stack([o, o % hubs], 1)])
    perm = torch.from_numpy(rng.permutation(n)).cuda()
    d = perm[d]
    d = d[torch.from_numpy(rng.permutation(d.shape[0])).cuda()].to(torch.int32).contiguous()
    deg = torch.bincount(d.flatten().long(), minlength=n)
    capped = int((deg >= 65535).sum())
    assert 0 < capped <= hubs and torch.unique(deg[deg >= 65535]).numel() < capped
    want = torch.empty(n, dtype=torch.int64, device="cuda")
    want[torch.argsort(deg, stable=True)] = torch.arange(n, device="cuda")
    pairs = want[d.long()]
    keys = torch.unique(pairs.min(1).values * n + pairs.max(1).values)
    rank, _, col = tc.build_csr(d, n)
    assert bool((rank.long() == want).all())
    assert bool((col.long() == keys % n).all())
