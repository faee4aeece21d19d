"""What a batch does to its replicas' lists: work items of full length while it is there, the estimate that sizes its
launches with them, short items again once it is gone, nothing if it could not be created, and no kernel on a list that
is still being built on another stream."""
import numpy as np
import pytest

import oracle
import synth
from _internals import load
from _nb import F, GpuSystem, max_atom_err, rel_rms

pytestmark = pytest.mark.gpu

RC, RL, BETA = 0.7, 0.8, 4.6


def _system(ctx=None, waters=700):
    return GpuSystem(synth.water_box(waters, synth.box_edge_for(waters), seed=waters), (8, 8), RL, ctx=ctx)


def _batch(s):
    import torch
    import paper_1306_1737_amd as mxn
    f = torch.zeros((s.box.n, 3), dtype=torch.float32, device=s.dev)
    return mxn.nb_batch_create(s.ctx, [s.grid], [s.lst], [s.xyzq], [f]), f


def _build(s, flags=0):
    import paper_1306_1737_amd as mxn
    mxn.nb_pairlist_build(s.ctx, s.grid, RL, -1.0, s.eo, s.ei, flags, s.lst)


def _items(s):
    import paper_1306_1737_amd as mxn
    return mxn.nb_list_info(s.lst)[1]


def test_estimate_of_full_items(tmp_path):
    import paper_1306_1737_amd as mxn
    internals = load(str(tmp_path))
    s = _system()
    try:
        short = _items(s)
        assert internals.list_est_items(s.lst) == short
        b, _ = _batch(s)
        full = _items(s)
        assert full < short
        assert internals.list_est_items(s.lst) == full
        mxn.nb_batch_free(b)
    finally:
        s.close()


def test_short_items_after_the_batch():
    import paper_1306_1737_amd as mxn
    s = _system()
    try:
        short = _items(s)
        b0, _ = _batch(s)
        b1, _ = _batch(s)
        full = _items(s)
        assert full < short
        mxn.nb_batch_free(b0)
        _build(s)
        assert _items(s) == full    # still bound to the other batch
        mxn.nb_batch_free(b1)
        _build(s)
        assert _items(s) == short
        b2, _ = _batch(s)
        mxn.nb_list_free(s.lst)     # lists may go before the batch
        s.lst = mxn.nb_pairlist_build(s.ctx, s.grid, RL, -1.0, s.eo, s.ei)
        mxn.nb_batch_free(b2)
        assert _items(s) == short
    finally:
        s.close()


def test_a_batch_that_is_not_created_changes_no_list():
    import paper_1306_1737_amd as mxn
    s = _system()
    try:
        short = _items(s)
        mxn.nb_grid_sort(s.ctx, s.box.box, s.xyzq, s.type, (8, 8), s.grid)   # the list is now older than its grid
        with pytest.raises(mxn.NbError) as e:
            _batch(s)
        assert e.value.status == mxn.NB_ERR_STATE
        assert _items(s) == short
        _build(s)
        assert _items(s) == short
    finally:
        s.close()


def test_created_while_a_list_is_built_on_another_stream():
    import torch
    import paper_1306_1737_amd as mxn
    s = _system()
    try:
        short = _items(s)
        mxn.nb_sync(s.ctx)
        a, b = torch.cuda.Stream(), torch.cuda.Stream()
        x = torch.randn(8192, 8192, device=s.dev, dtype=torch.bfloat16)
        torch.cuda.synchronize()
        with torch.cuda.stream(a):   # some 50 ms of work before the build
            for _ in range(50):
                torch.mm(x, x)
        mxn.nb_set_stream(s.ctx, a)
        _build(s, mxn.NB_LIST_ASYNC)
        mxn.nb_set_stream(s.ctx, b)
        batch, f = _batch(s)
        torch.cuda.synchronize()
        assert _items(s) < short
        e = torch.zeros((1, 2), dtype=torch.float64, device=s.dev)
        mxn.nb_batch_forces(s.ctx, batch, mxn.make_params(RC, BETA, F, s.lj), mxn.NB_ENERGY, e)
        mxn.nb_sync(s.ctx)
        fr, er, _ = oracle.forces(s.box.xyz, s.box.q, s.box.type, s.box.box, s.box.excl_off, s.box.excl_idx,
                                  synth.lj_table_spce(), RC, BETA, F)
        f = f.cpu().numpy().astype(np.float64)
        assert rel_rms(f, fr) <= 1e-5 and max_atom_err(f, fr) <= 1e-4
        np.testing.assert_allclose(e.cpu().numpy()[0], er, rtol=1e-5, atol=1e-5 * np.abs(er).max())
        mxn.nb_batch_free(batch)
        torch.cuda.synchronize()
    finally:
        s.close()
