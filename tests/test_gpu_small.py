"""Small graphs on the bit matrix (heuristic and learned selection, at most 16384 vertices and 2^17 pairs)
against the oracle and against the general pipeline, at the edges of the matrix's row widths (4096, 8192,
16384 vertices), of a build block's rows (16, 32, 64) and of the size rule."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

MAX_N, MAX_PAIRS = 16384, 1 << 17


@pytest.fixture(scope="module")
def tc():
    import paper_1804_06926_amd as tc
    from paper_1804_06926_amd import selector
    assert selector.load_default()
    return tc


def _dirty(n, pairs, seed):
    """Skewed endpoints with loops and repeats in both directions, every id reachable."""
    rng = np.random.Generator(np.random.PCG64(seed))
    e = np.minimum((rng.random((pairs, 2)) ** 3 * n).astype(np.int32), n - 1)
    e[0] = (0, n - 1)
    return e


GRAPHS = {
    "one_vertex": lambda: (np.zeros((3, 2), dtype=np.int32), 1),
    "one_pair": lambda: (np.array([[1, 0]], dtype=np.int32), 2),
    "triangle": lambda: (np.array([[0, 1], [2, 1], [0, 2], [2, 0]], dtype=np.int32), 3),
    "n16": lambda: (_dirty(16, 100, 1), 16),
    "n17": lambda: (_dirty(17, 65, 2), 17),
    "n64": lambda: (graphgen.complete(64), 64),
    "star": lambda: (graphgen.star(16383), 16384),
    "complete_512": lambda: (graphgen.complete(512), 512),
    "n4095": lambda: (_dirty(4095, 30001, 3), 4095),
    "n4096": lambda: (_dirty(4096, 8193, 4), 4096),
    "n4097": lambda: (_dirty(4097, 40000, 5), 4097),
    "n8192": lambda: (_dirty(8192, MAX_PAIRS, 6), 8192),
    "n8193": lambda: (_dirty(8193, 70001, 7), 8193),
    "n16383": lambda: (_dirty(16383, 100003, 8), 16383),
    "at_rule": lambda: (_dirty(MAX_N, MAX_PAIRS, 9), MAX_N),
    "pairs_past_rule": lambda: (_dirty(MAX_N, MAX_PAIRS + 1, 9), MAX_N),
    "vertices_past_rule": lambda: (_dirty(MAX_N + 1, MAX_PAIRS, 9), MAX_N + 1),
    "isolated": lambda: (np.array([[5, 9000], [9000, 12000], [12000, 5]], dtype=np.int32), 16000),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_small_counts(tc, name):
    import torch
    e, n = GRAPHS[name]()
    e = np.ascontiguousarray(e, dtype=np.int32)
    T, t = oracle.count_triangles(e, n, per_vertex=True)
    d = torch.from_numpy(e).cuda()
    ref = tc.clustering(d, n, per_vertex=True, select=tc.FORCE_MERGE)   # the pipeline
    for sel in (tc.SELECT_HEURISTIC, tc.SELECT_LEARNED):
        Tx, tx = tc.count_triangles(d, n, per_vertex=True, select=sel)
        assert Tx == T
        np.testing.assert_array_equal(tx.cpu().numpy().astype(np.uint64), t)
        got = tc.clustering(d, n, per_vertex=True, select=sel)
        assert got[1:4] == ref[1:4]
        np.testing.assert_array_equal(got[0].cpu().numpy(), ref[0].cpu().numpy())
        np.testing.assert_array_equal(got[4].cpu().numpy(), ref[4].cpu().numpy())
        # queued: T, status and t[v]
        res = torch.full((2,), -1, dtype=torch.int64, device="cuda")
        pv = torch.full((n,), -1, dtype=torch.int64, device="cuda")
        tc.count_triangles_async(d, n, result=res, per_vertex=pv, select=sel)
        assert res.cpu().tolist() == [T, 0]
        np.testing.assert_array_equal(pv.cpu().numpy().astype(np.uint64), t)


@pytest.mark.parametrize("name", ["n17", "n4095", "n8193", "at_rule", "star", "complete_512", "isolated"])
def test_small_statistics_equal_the_pipeline(tc, name):
    """Every field of the last call's statistics is what the pipeline reports (run with stage times,
    which are the pipeline's)."""
    import torch
    e, n = GRAPHS[name]()
    d = torch.from_numpy(np.ascontiguousarray(e, dtype=np.int32)).cuda()
    for sel in (tc.SELECT_HEURISTIC, tc.SELECT_LEARNED):
        tc.count_triangles(d, n, select=sel, timing=True)
        ref, ref_f = tc.last_stats(), tc.bucket_features()
        tc.count_triangles(d, n, select=sel)
        got, got_f = tc.last_stats(), tc.bucket_features()
        for k in ref:
            np.testing.assert_array_equal(got[k], ref[k], err_msg=k)
        np.testing.assert_array_equal(got_f, ref_f)


@pytest.mark.parametrize("pair", [(3, 4096), (-1, 3), (4096, 4096), (2, 2**31 - 1), (-2**31, 0)])
def test_small_range_errors(tc, pair):
    import torch
    e = np.concatenate([_dirty(4096, 5000, 3), np.array([pair], dtype=np.int64).astype(np.int32)])
    d = torch.from_numpy(np.ascontiguousarray(e)).cuda()
    with pytest.raises(tc.TCError) as ei:
        tc.count_triangles(d, 4096)
    assert ei.value.status == 2
    res = torch.full((2,), -1, dtype=torch.int64, device="cuda")
    tc.count_triangles_async(d, 4096, result=res)
    assert int(res[1]) == 2
    assert tc.count_triangles(d[:5000], 4096) == oracle.count_triangles(e[:5000], 4096)


def test_small_graph_in_a_smaller_workspace_and_under_capture(tc):
    """A workspace too small for the matrix still counts (the pipeline needs less), and a captured call
    replays with other inputs in the same buffer and other work between."""
    import ctypes
    import torch
    n, E = 16000, 20000
    a, b = _dirty(n, E, 11), _dirty(n, E, 12)
    Ta, Tb = oracle.count_triangles(a, n), oracle.count_triangles(b, n)
    d = torch.from_numpy(a).cuda()
    lib = tc._lib._load()
    full = tc.workspace_size(E, n)
    assert full > 16000 * 2048   # the matrix
    # the pipeline's own need is far below the matrix: 8 MB here
    ws = torch.empty(8 << 20, dtype=torch.uint8, device="cuda")
    ctx, _ = tc._lib._ctx(d.device)
    o, count = tc._lib.Options(), ctypes.c_uint64()
    assert lib.tc_count_triangles(ctx, d.data_ptr(), E, n, ws.data_ptr(), ws.numel(), ctypes.byref(o),
                                  ctypes.byref(count), None) == 0
    assert count.value == Ta
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    res = torch.zeros(2, dtype=torch.int64, device="cuda")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        tc.count_triangles_async(d, n, result=res, workspace=ws)   # the context of this stream
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            tc.count_triangles_async(d, n, result=res, workspace=ws)
    for x, T in ((a, Ta), (b, Tb), (a, Ta), (b, Tb)):
        d.copy_(torch.from_numpy(x))
        res.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert res.cpu().tolist() == [T, 0]
        assert tc.count_triangles(torch.from_numpy(b).cuda(), n) == Tb
