"""Run sorts at the edges of the batches of short runs (64 positions, 64 runs, 26 low bits) and of the lengths that one
wave sorts (1024)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LENGTHS = {
    "full_batches": [64] * 40 + [32, 32] * 40 + [63, 1] * 40 + [2] * 640 + [1] * 640 + [21, 21, 22] * 30,
    "one_over": [64, 1] * 60 + [33, 32] * 60 + [1] * 63 + [2] * 33 + [65] * 3 + [1, 64, 65] * 20,
    "wave_limit": [1023, 1, 1024, 1, 1025, 63, 64, 1024, 1025, 65] * 4,
    "past_the_tile": ([1] * 4095 + [1024]) * 3 + [3072, 1, 1023] + ([1] * 4094 + [1025]) * 3 + [64] * 64 + [1] * 4033 + [64],
    "skips": [65] * 63 + [1] + [65] * 64 + [2, 700, 3] * 30 + [65] * 130 + [5],
}


@pytest.mark.parametrize("name", sorted(LENGTHS))
@pytest.mark.parametrize("shift", [9, 24, 26, 27])
def test_runs(name, shift):
    import torch
    import paper_1804_06926_amd as tc
    rng = np.random.Generator(np.random.PCG64(shift))
    lens = np.asarray(LENGTHS[name], dtype=np.int64)
    high = np.repeat(np.cumsum(rng.integers(1, 4, lens.size)), lens).astype(np.uint64)
    low = rng.integers(0, 1 << shift, high.size, dtype=np.uint64)
    low[rng.random(high.size) < 0.2] = np.uint64((1 << shift) - 1)   # repeated, and all ones
    keys = (high << np.uint64(shift)) | low
    d = torch.from_numpy(keys.view(np.int64).copy()).to("cuda:0")
    tc.sort_runs_u64(d, shift)
    np.testing.assert_array_equal(d.cpu().numpy().view(np.uint64), np.sort(keys))


@pytest.mark.parametrize("name", sorted(LENGTHS))
def test_rows_of_a_graph(name):
    """The same lengths as out-lists with repeated pairs: the exported CSR is free of them and sorted."""
    import torch
    import paper_1804_06926_amd as tc
    rng = np.random.Generator(np.random.PCG64(len(name)))
    lens = np.asarray(LENGTHS[name], dtype=np.int64)
    n = lens.size + 3000
    e = np.stack([np.repeat(np.arange(lens.size), lens), rng.integers(0, n, lens.sum())], 1).astype(np.int32)
    d = torch.from_numpy(np.concatenate([e, e[::3]])).cuda()
    rank, off, col = tc.build_csr(d, n)
    p = rank.long()[d[d[:, 0] != d[:, 1]].long()]
    keys = torch.unique(p.min(1).values * n + p.max(1).values)
    assert torch.equal(off[1:].long(), torch.cumsum(torch.bincount(keys // n, minlength=n), 0))
    assert torch.equal(col.long(), keys % n)
