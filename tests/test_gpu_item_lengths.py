"""Lists with work items of one, two and four passes: forces and energies against the oracle, items covering every entry
once, asynchronous rebuilds, and a batch bound to them with and without a topology."""
import numpy as np
import pytest

import oracle
import synth
from _nb import F, GpuSystem, max_atom_err, rel_rms

pytestmark = pytest.mark.gpu

RC, RL, BETA = 0.7, 0.8, 4.6


def _ref(box):
    return oracle.forces(box.xyz, box.q, box.type, box.box, box.excl_off, box.excl_idx, synth.lj_table_spce(), RC, BETA, F)


def _close(f, e, ref):
    assert rel_rms(f, ref[0]) <= 1e-5 and max_atom_err(f, ref[0]) <= 1e-4
    np.testing.assert_allclose(e, ref[1], rtol=1e-5, atol=1e-5 * np.abs(ref[1]).max())


@pytest.mark.parametrize("shape", [(4, 4), (4, 8), (8, 4), (8, 8)])
@pytest.mark.parametrize("waters", [200, 2000, 4000, 9000])
def test_lengths(shape, waters):
    import paper_1306_1737_amd as mxn
    box = synth.water_box(waters, synth.box_edge_for(waters), seed=waters)
    ref = _ref(box)
    s = GpuSystem(box, shape, RL)
    try:
        entries, items = mxn.nb_list_info(s.lst)
        full = 256 // shape[1]
        assert items * full >= entries and items <= entries
        if waters == 200:
            assert items >= entries / (full // 4)       # one pass each
        for flags in (0, mxn.NB_LIST_ASYNC):
            mxn.nb_pairlist_build(s.ctx, s.grid, RL, -1.0, s.eo, s.ei, flags, s.lst)
            f, e, _ = s.forces(RC, BETA, mxn.NB_ENERGY)
            _close(f, e, ref)
            assert mxn.nb_list_info(s.lst) == (entries, items)
    finally:
        s.close()


@pytest.mark.parametrize("topology", [False, True])
def test_batch_of_short_lists(topology):
    import torch
    import paper_1306_1737_amd as mxn
    boxes = [synth.water_box(w, synth.box_edge_for(w), seed=w) for w in (200, 700, 3000)]
    ctx = mxn.nb_create(0)
    sys_ = [GpuSystem(b, (8, 8), RL, ctx=ctx) for b in boxes]
    try:
        lens = [mxn.nb_list_info(s.lst) for s in sys_]
        fs = [torch.zeros((b.n, 3), dtype=torch.float32, device="cuda:0") for b in boxes]
        e = torch.zeros((len(boxes), 2), dtype=torch.float64, device="cuda:0")
        b = mxn.nb_batch_create(ctx, [s.grid for s in sys_], [s.lst for s in sys_], [s.xyzq for s in sys_], fs)
        if topology:
            mxn.nb_batch_bind_topology(b, [s.type for s in sys_], [s.eo for s in sys_], [s.ei for s in sys_])
        mxn.nb_sync(ctx)
        for s, was in zip(sys_, lens):   # the same entries in fewer items
            now = mxn.nb_list_info(s.lst)
            assert now[0] == was[0] and now[1] <= was[1]
        p = mxn.make_params(RC, BETA, F, sys_[0].lj)
        for k in range(2):
            mxn.nb_batch_forces(ctx, b, p, mxn.NB_ENERGY, e)
            mxn.nb_sync(ctx)
            for f, en, box in zip(fs, e.cpu().numpy(), boxes):
                _close(f.cpu().numpy().astype(np.float64), en, _ref(box))
            if not topology:
                break
            mxn.nb_batch_rebuild(ctx, b)
        f1, e1, _ = sys_[0].forces(RC, BETA, mxn.NB_ENERGY)   # the replica's own list still serves single calls
        _close(f1, e1, _ref(boxes[0]))
        mxn.nb_batch_free(b)
    finally:
        for s in sys_:
            mxn.nb_list_free(s.lst)
            mxn.nb_grid_free(s.grid)
        mxn.nb_destroy(ctx)
