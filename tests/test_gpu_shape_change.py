"""Handles that change their cluster shape between builds: the grid re-sorted in another shape, the list rebuilt on it
(an asynchronous build included, which has to reserve anew) and a pruned list; lists bit-exact and forces against the
oracle.  A batch whose replica was re-sorted in another shape is refused."""
import numpy as np
import pytest

import oracle
import synth
from _nb import F, GpuSystem, default_rbb, max_atom_err, rel_rms

pytestmark = pytest.mark.gpu

RC, RL, BETA = 0.6, 0.62, 5.2


@pytest.mark.parametrize("first,then", [((8, 8), (8, 4)), ((8, 4), (8, 8)), ((4, 8), (8, 8)), ((8, 8), (4, 8)),
                                        ((4, 8), (8, 4)), ((4, 4), (8, 8)), ((8, 8), (4, 4))])
@pytest.mark.parametrize("asynchronous", [True, False])
def test_rebuilt_in_another_shape(first, then, asynchronous):
    import paper_1306_1737_amd as mxn
    box = synth.water_box(1500, synth.box_edge_for(1500), seed=15)
    fr, er, _ = oracle.forces(box.xyz, box.q, box.type, box.box, box.excl_off, box.excl_idx, synth.lj_table_spce(), RC,
                              BETA, F)
    s = GpuSystem(box, first, RL)
    inner = None
    try:
        for shape in (first, then, first, then):
            mxn.nb_grid_sort(s.ctx, box.box, s.xyzq, s.type, shape, s.grid)
            mxn.nb_pairlist_build(s.ctx, s.grid, RL, -1.0, s.eo, s.ei, mxn.NB_LIST_ASYNC if asynchronous else 0, s.lst)
            inner = mxn.nb_pairlist_prune(s.ctx, s.lst, s.xyzq, RL, inner)
            mxn.nb_sync(s.ctx)
            og = oracle.grid_sort(box.xyz, box.box, *shape)
            ref = oracle.pairlist(og, box.box, RL, default_rbb(box, shape, RL), box.excl_off, box.excl_idx)
            got = mxn.nb_list_export_canonical(s.lst)
            for k in ("ci", "shift", "cj", "mask"):
                np.testing.assert_array_equal(got[k], ref[k])
            whole = s.lst
            for lst in (whole, inner):
                s.lst = lst
                f, e, _ = s.forces(RC, BETA, mxn.NB_ENERGY)
                assert rel_rms(f, fr) <= 1e-5 and max_atom_err(f, fr) <= 1e-4
                np.testing.assert_allclose(e, er, rtol=1e-5, atol=1e-5 * np.abs(er).max())
            s.lst = whole
    finally:
        if inner is not None:
            mxn.nb_list_free(inner)
        s.close()


def test_batch_refuses_another_shape():
    """Every call that would run the batch's kernels, before and after a capture."""
    import torch
    import paper_1306_1737_amd as mxn
    box = synth.water_box(400, synth.box_edge_for(400), seed=4)
    s = GpuSystem(box, (8, 8), RL)
    try:
        f = torch.zeros((box.n, 3), dtype=torch.float32, device=s.dev)
        p = mxn.make_params(RC, BETA, F, s.lj)
        b = mxn.nb_batch_create(s.ctx, [s.grid], [s.lst], [s.xyzq], [f])
        mxn.nb_batch_bind_topology(b, [s.type], [s.eo], [s.ei])
        mxn.nb_batch_capture_cycle(s.ctx, b, 1, p, 0)
        mxn.nb_batch_replay(s.ctx, b)
        mxn.nb_sync(s.ctx)
        first = f.clone()
        mxn.nb_grid_sort(s.ctx, box.box, s.xyzq, s.type, (8, 4), s.grid)
        mxn.nb_pairlist_build(s.ctx, s.grid, RL, -1.0, s.eo, s.ei, 0, s.lst)
        for call in (lambda: mxn.nb_batch_forces(s.ctx, b, p, 0), lambda: mxn.nb_batch_rebuild(s.ctx, b),
                     lambda: mxn.nb_batch_replay(s.ctx, b), lambda: mxn.nb_batch_capture(s.ctx, b, p, 0),
                     lambda: mxn.nb_batch_capture_cycle(s.ctx, b, 1, p, 0)):
            with pytest.raises(mxn.NbError) as e:
                call()
            assert e.value.status == mxn.NB_ERR_STATE
        mxn.nb_sync(s.ctx)
        assert (f == first).all()
        mxn.nb_grid_sort(s.ctx, box.box, s.xyzq, s.type, (8, 8), s.grid)   # back in its shape it runs again
        mxn.nb_pairlist_build(s.ctx, s.grid, RL, -1.0, s.eo, s.ei, 0, s.lst)
        mxn.nb_batch_forces(s.ctx, b, p, 0)
        mxn.nb_sync(s.ctx)
        fr, _, _ = oracle.forces(box.xyz, box.q, box.type, box.box, box.excl_off, box.excl_idx, synth.lj_table_spce(), RC,
                                 BETA, F)
        for g in (f, first):
            g = g.cpu().numpy().astype(np.float64)
            assert rel_rms(g, fr) <= 1e-5 and max_atom_err(g, fr) <= 1e-4
        mxn.nb_batch_free(b)
    finally:
        s.close()
