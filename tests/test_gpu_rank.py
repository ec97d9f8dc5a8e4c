"""The degree order of vertices about the highest degree that is sorted on (65534), and the offsets of the oriented
rows for vertex counts about one scan step (2048) and one step for each of 1024 blocks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tc():
    import paper_1804_06926_amd as tc
    return tc


def _check(tc, e, n):
    import torch
    d = torch.from_numpy(np.ascontiguousarray(e, dtype=np.int32)).cuda()
    keep = d[:, 0] != d[:, 1]
    deg = torch.bincount(d[keep].flatten().long(), minlength=n)
    order = torch.argsort(deg, stable=True)
    want = torch.empty(n, dtype=torch.int64, device="cuda")
    want[order] = torch.arange(n, device="cuda")
    pairs = want[d[keep].long()]
    keys = torch.unique(pairs.min(1).values * n + pairs.max(1).values)
    rank, off, col = tc.build_csr(d, n)
    assert bool((rank.long() == want).all())
    row = torch.bincount(keys // n, minlength=n)
    assert int(off[0]) == 0 and bool((off[1:].long() == torch.cumsum(row, 0)).all())
    assert bool((col.long() == keys % n).all())


@pytest.mark.parametrize("n", [900, 70_001, 5_000_000])
@pytest.mark.parametrize("degrees", [(65535,), (65534, 65535, 65536, 65535, 65534), (65536, 131072, 65535, 70000, 65536, 65535)])
def test_rank_of_the_highest_degrees(tc, n, degrees):
    rng = np.random.Generator(np.random.PCG64(n + len(degrees)))
    hubs = rng.choice(n, size=len(degrees), replace=False)
    leaves = np.setdiff1d(np.arange(min(n, 100_000)), hubs)
    parts = [np.stack([np.full(k, h), rng.choice(leaves, size=k)], 1) for h, k in zip(hubs, degrees)]
    parts.append(np.stack([hubs, hubs], 1))   # loops count for no degree
    e = np.concatenate(parts)
    flip = rng.random(len(e)) < 0.5
    e[flip] = e[flip][:, ::-1]
    _check(tc, rng.permutation(e), n)


@pytest.mark.parametrize("n", [2, 2047, 2048, 2049, 4096, (1 << 21) - 1, 1 << 21, (1 << 21) + 1, (1 << 22) + 2049])
def test_offsets_about_the_scan_steps(tc, n):
    rng = np.random.Generator(np.random.PCG64(n))
    e = rng.integers(0, n, size=(max(n // 2, 1) + 777, 2))
    _check(tc, e, n)
