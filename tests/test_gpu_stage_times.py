"""The stage times name the kernels that ran in them."""
import pytest

import graphgen

pytestmark = pytest.mark.gpu


def test_merge_stage_is_the_merge_kernel_alone():
    """With the bitmap strategy forced, merge path and binary search have no tiles, and their stages are two empty
    launches of like size. The 16-bit columns of 2^26 pairs (0.4 GB moved, 80 us at the copy's rate) and the hub
    kernels' ranges belong to the layout of the tiles before them."""
    import torch
    import paper_1804_06926_amd as tc
    d = torch.from_numpy(graphgen.rmat(22, 16, seed=6)).cuda()
    runs = [tc.count_triangles(d, 1 << 22, select=tc.FORCE_BITMAP, timing=True)[1] for _ in range(6)][1:]
    merge, bsearch = (sorted(r[k] for r in runs)[2] for k in ("isect_merge", "isect_bsearch"))
    assert merge < bsearch + 0.03, (merge, bsearch)
