"""A given workspace serves every call of equal or smaller sizes, also one whose small graph's bit matrix it has no
room for; and calls without a matrix allocate none."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

LARGE, SMALL = (150_000, 20_000), (90_000, 16_000)   # pairs, vertices: the smaller one has a matrix


@pytest.fixture(scope="module")
def tc():
    import paper_1804_06926_amd as tc
    return tc


@pytest.fixture(scope="module")
def graph():
    import torch
    pairs, n = SMALL
    rng = np.random.Generator(np.random.PCG64(5))
    e = np.minimum((rng.random((pairs, 2)) ** 3 * n).astype(np.int32), n - 1)
    return torch.from_numpy(e).cuda(), n, oracle.count_triangles(e, n)


def _calls(tc, d, n, ws):
    yield "count", lambda: tc.count_triangles(d, n, workspace=ws)
    yield "count t", lambda: tc.count_triangles(d, n, per_vertex=True, workspace=ws)[0]
    yield "timing", lambda: tc.count_triangles(d, n, workspace=ws, timing=True)[0]
    yield "async", lambda: int(tc.count_triangles_async(d, n, workspace=ws)[0])
    yield "clustering", lambda: tc.clustering(d, n, workspace=ws)[1]
    yield "support", lambda: tc.edge_support(d, n, workspace=ws)[2]
    yield "edge counts", lambda: tc.edge_counts(d, n, workspace=ws)[2]
    for form in ("filtered", "matrix_upper"):
        yield form, lambda: tc.count_triangles_formulation(d, n, form, workspace=ws)[0]
    yield "choices", lambda: tc.profile_choices(d, n, np.full(256, 255, np.uint8), repeats=1, workspace=ws)[2]
    yield "csr", lambda: tc.build_csr(d, n, workspace=ws)
    yield "buckets", lambda: tc.profile_buckets(d, n, repeats=1, workspace=ws)
    yield "selected", lambda: tc.profile_selected(d, n, repeats=1, workspace=ws)


def test_smaller_call_in_a_larger_calls_workspace(tc, graph):
    import torch
    d, n, T = graph
    ws = torch.empty(tc.workspace_size(*LARGE), dtype=torch.uint8, device="cuda")
    assert ws.numel() < tc.workspace_size(*SMALL)
    for name, call in _calls(tc, d, n, ws):
        got = call()
        assert not isinstance(got, int) or got == T, name
    for form in ("full", "matrix"):   # these need more than a plain count
        torch.cuda.synchronize()
        nb = tc.workspace_size(*LARGE) + 8 * LARGE[0] + 4 * (LARGE[1] + 1) + 512
        big = torch.empty(nb, dtype=torch.uint8, device="cuda")
        assert tc.count_triangles_formulation(d, n, form, workspace=big)[0] == T


def test_too_small_a_workspace_is_refused(tc, graph):
    import torch
    d, n, _ = graph
    least = tc._lib._workspace_size_min(*SMALL)
    assert least < tc.workspace_size(*LARGE)
    ws = torch.empty(least - 1, dtype=torch.uint8, device="cuda")
    for name, call in _calls(tc, d, n, ws):
        with pytest.raises(tc.TCError) as ei:
            call()
        assert ei.value.status == 3, name


def test_calls_without_a_matrix_allocate_none(tc):
    import torch
    d = torch.tensor([[0, 1], [1, 2], [2, 0]], dtype=torch.int32, device="cuda")
    n = 16_000
    assert tc.workspace_size(3, n) > n * 2048   # the matrix
    held = tc._lib._workspaces
    kept = dict(held)
    held.clear()
    try:
        assert tc.edge_support(d, n)[2] == tc.edge_counts(d, n)[2] == 1
        tc.build_csr(d, n)
        tc.profile_buckets(d, n, repeats=1)
        tc.profile_selected(d, n, repeats=1)
        assert tc.count_triangles(d, n, select=tc.FORCE_MERGE) == 1
        assert tc.count_triangles_formulation(d, n, "full")[0] == 1
        assert max(w.numel() for w in held.values()) < 4 << 20
        assert tc.count_triangles(d, n) == 1
        assert max(w.numel() for w in held.values()) == tc.workspace_size(3, n)
    finally:
        held.update(kept)
