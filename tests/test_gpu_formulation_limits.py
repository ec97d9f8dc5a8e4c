"""The whole-row formulations past 2^30 kept edges, where positions in the symmetric adjacency pass 2^31."""
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(600)]


@pytest.fixture(scope="module")
def tc():
    import paper_1804_06926_amd as tc
    return tc


def test_symmetric_positions_past_2_31(tc):
    """The circulant graph on n = 2^25 + 3 vertices where i is joined to i + 1 .. i + 33: 33 n = 1,107,296,355 edges,
    so that the rows of the last million vertices lie past position 2^31. A triangle is a vertex and two of the 33
    distances after it: T = n C(33, 2)."""
    import torch
    n, k = (1 << 25) + 3, 33
    T = n * (k * (k - 1) // 2)
    i = torch.arange(n, device="cuda", dtype=torch.int32)
    d = torch.empty((n, k, 2), dtype=torch.int32, device="cuda")
    for j in range(k):
        d[:, j, j % 2] = i
        d[:, j, 1 - j % 2] = torch.where(i >= n - 1 - j, i - (n - 1 - j), i + (j + 1))   # (i + j + 1) mod n
    d = d.view(-1, 2)
    assert d.shape[0] > 1 << 30
    print(f"[formulation limits] E={d.shape[0]} n={n}", flush=True)
    for form, multiple, sel in (("full", 3, tc.FORCE_MERGE), ("full", 3, tc.FORCE_BITMAP),
                                ("matrix", 2, tc.FORCE_BSEARCH), ("matrix", 2, tc.FORCE_BITMAP)):
        got = tc.count_triangles_formulation(d, n, form, select=sel)
        print(f"[formulation limits] {form} {sel}: {got}", flush=True)
        assert got == (T, multiple * T)
    del d
    torch.cuda.empty_cache()
    tc._lib._workspaces.clear()
