"""Boxes thinner than a grid column, where the columns hold far less than a cluster each: the grid's storage follows the
particles, not the box's extent along z, and sort and list are the oracle's.  Boxes so flat that the columns outnumber an int are
refused, and a grid that was refused a sort still serves its list."""
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


@pytest.mark.parametrize("box", [(100.0, 100.0, 1e-9), (100.0, 100.0, 1e-12), (100.0, 100.0, 1e-30), (1e-200, 1e-200, 1.0)])
def test_too_many_columns(box):
    import paper_1306_1737_amd as mxn
    import synth
    from _nb import GpuSystem
    w = synth.water_box(300, synth.box_edge_for(300), seed=2)
    s = GpuSystem(w, (8, 8), 0.7)
    try:
        first = s.forces(0.65, 4.6, mxn.NB_ENERGY)
        for grid in (s.grid, None):
            with pytest.raises(mxn.NbError) as e:
                mxn.nb_grid_sort(s.ctx, box, s.xyzq, s.type, (8, 4), grid)
            assert e.value.status == mxn.NB_ERR_ARG
        for a, b in zip(first, s.forces(0.65, 4.6, mxn.NB_ENERGY)):
            np.testing.assert_array_equal(a, b)
    finally:
        s.close()
