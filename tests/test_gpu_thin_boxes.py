"""Boxes thinner than a grid column, where the columns hold far less than a cluster each: the grid's storage follows the
particles, not the box's extent along z, and sort and list are the oracle's."""
import numpy as np
import pytest

import oracle
from test_gpu_search_forms import SHAPES, _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("box,n", [((2e-4, 300.0, 300.0), 3000), ((1e-3, 1e-3, 9e4), 2500)])
def test_storage_and_list(shape, box, n):
    import torch
    import paper_1306_1737_amd as mxn
    rng = np.random.default_rng(n)
    box = np.array(box)
    xyz = (rng.uniform(0.0, 1.0, (n, 3)) * box).astype(np.float32)
    xyz[n // 2:] = xyz[:n - n // 2] + rng.uniform(-6e-5, 6e-5, (n - n // 2, 3)).astype(np.float32)   # close pairs
    dev = torch.device("cuda:0")
    ctx = mxn.nb_create(0)
    try:
        xyzq = np.zeros((n, 4), np.float32)
        xyzq[:, :3] = xyz
        g = mxn.nb_grid_sort(ctx, box, torch.from_numpy(xyzq).to(dev), torch.zeros(n, dtype=torch.int32, device=dev), shape)
        mxn.nb_sync(ctx)
        got = mxn.nb_grid_export(g)
        og = oracle.grid_sort(xyz, box, *shape)
        np.testing.assert_array_equal(got["perm"], og["perm"])
        # slots: positions twice, type, particle, image, boxes (at most 2 x 32 bytes for each 4 slots); columns: counts,
        # starts, extents; and an index of some four bins (32 bytes) for each j-cluster of the capacity
        slots = n + got["info"]["nx"] * got["info"]["ny"] * max(shape)
        assert sum(mxn.nb_memory_info(ctx)) <= 128 * slots + 65536
        mxn.nb_grid_free(g)
    finally:
        mxn.nb_destroy(ctx)
    _check(xyz, box, shape, 9e-5, -1.0, np.zeros(n + 1), np.zeros(1))
