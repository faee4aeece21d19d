"""A synchronous rebuild moves a list's storage only when its entries outgrow it, also where the rebuilt list would be
short enough for shorter work items: force calls captured before the rebuild then still run on the list's buffers."""
import numpy as np
import pytest

import oracle
import synth
from _nb import F, GpuSystem, max_atom_err, rel_rms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(8, 4), (8, 8)])
def test_rebuilt_with_fewer_entries(shape):
    import torch
    import paper_1306_1737_amd as mxn
    rc, beta = 0.6, 5.2
    box = synth.water_box(4000, synth.box_edge_for(4000), seed=44)
    s = GpuSystem(box, shape, 1.3)
    fresh = None
    try:
        full = 256 // shape[1]
        n0 = mxn.nb_list_info(s.lst)
        assert n0[1] < n0[0] / (full // 2)   # items of full length
        p = mxn.make_params(rc, beta, F, s.lj)
        f = torch.zeros((box.n, 3), dtype=torch.float32, device=s.dev)
        e = torch.zeros(2, dtype=torch.float64, device=s.dev)
        mxn.nb_forces(s.ctx, s.grid, s.lst, s.xyzq, p, mxn.NB_ENERGY, f, e)
        mxn.nb_sync(s.ctx)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            mxn.nb_set_stream(s.ctx)
            mxn.nb_forces(s.ctx, s.grid, s.lst, s.xyzq, p, mxn.NB_ENERGY, f, e)
        mxn.nb_set_stream(s.ctx)
        held = mxn.nb_memory_info(s.ctx)
        mxn.nb_pairlist_build(s.ctx, s.grid, 0.7, -1.0, s.eo, s.ei, 0, s.lst)
        mxn.nb_sync(s.ctx)
        assert mxn.nb_list_info(s.lst)[0] < n0[0]
        assert mxn.nb_memory_info(s.ctx) == held
        fr, er, _ = oracle.forces(box.xyz, box.q, box.type, box.box, box.excl_off, box.excl_idx, synth.lj_table_spce(),
                                  rc, beta, F, mode="binned")
        for _ in range(3):
            f.fill_(float("nan"))
            graph.replay()
            fe, ee, _ = s.forces(rc, beta, mxn.NB_ENERGY)   # eager work between the replays
            torch.cuda.synchronize()
            for fk, ek in ((f.cpu().numpy().astype(np.float64), e.cpu().numpy()), (fe, ee)):
                assert rel_rms(fk, fr) <= 1e-5 and max_atom_err(fk, fr) <= 1e-4
                np.testing.assert_allclose(ek, er, rtol=1e-5)
        assert mxn.nb_memory_info(s.ctx) == held
        # a list that starts with these entries does take short items
        fresh = mxn.nb_pairlist_build(s.ctx, s.grid, 0.7, -1.0, s.eo, s.ei)
        n1 = mxn.nb_list_info(fresh)
        assert n1[1] > mxn.nb_list_info(s.lst)[1] and n1[0] == mxn.nb_list_info(s.lst)[0]
    finally:
        if fresh is not None:
            mxn.nb_list_free(fresh)
        s.close()


def test_flip_within_the_storage():
    """Storage sized for short items serves both lengths: a longer list in it takes full items, a shorter one short ones."""
    import paper_1306_1737_amd as mxn
    box = synth.water_box(300, synth.box_edge_for(300), seed=9)
    s = GpuSystem(box, (8, 8), 0.65)
    try:
        n0, held = mxn.nb_list_info(s.lst), mxn.nb_memory_info(s.ctx)
        for rlist in (0.6, 0.65):
            mxn.nb_pairlist_build(s.ctx, s.grid, rlist, -1.0, s.eo, s.ei, 0, s.lst)
            mxn.nb_sync(s.ctx)
            assert mxn.nb_memory_info(s.ctx) == held
        assert mxn.nb_list_info(s.lst) == n0
    finally:
        s.close()
