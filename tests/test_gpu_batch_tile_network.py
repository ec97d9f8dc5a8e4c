"""A captured batch follows the tile network: setting or removing it between two calls of one shape."""
import numpy as np
import pytest

import graphgen

pytestmark = pytest.mark.gpu


def test_captured_batch_follows_the_tile_network(tc):
    import torch
    from paper_1804_06926_amd import _lib, selector
    e, off, nv = graphgen.chung_lu_batch(32, 1e3, 3e4, seed=23)
    d = torch.from_numpy(e).cuda()
    half = np.zeros(_lib.SELECTOR_NUM_PARAMS, dtype=np.float32)
    half[-3] = 1.0   # the logit of the first class alone: half the rule's in-edges per tile
    double = np.zeros_like(half)
    double[-1] = 1.0

    def chunks(tile, graph):
        tc.selector_set_tile_params(tile)
        tc.count_triangles_batch(d, off, nv, select=tc.SELECT_LEARNED, graph=graph)
        return tc.last_stats()["bucket_chunk"]

    selector.load_default()
    try:
        want = [chunks(t, False) for t in (half, None, double)]
        assert np.any(want[0] != want[1]) and np.any(want[1] != want[2])
        for t, w in ((half, want[0]), (None, want[1]), (double, want[2]), (None, want[1]), (half, want[0]),
                     (half, want[0])):
            np.testing.assert_array_equal(chunks(t, True), w)
    finally:
        selector.load_default()


@pytest.fixture(scope="module")
def tc():
    import paper_1804_06926_amd as tc
    return tc
