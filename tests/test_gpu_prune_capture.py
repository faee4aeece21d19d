"""A captured prune into a handle that last held a larger list, replayed with other work between the replays: the counters
it clears in the graph start from zero every time."""
import numpy as np
import pytest

import oracle
import synth
from _nb import F, GpuSystem, max_atom_err, rel_rms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(8, 4), (8, 8)])
def test_replays(shape):
    import torch
    import paper_1306_1737_amd as mxn
    rc, rl, beta = 0.6, 0.7, 5.2
    big, box = (synth.water_box(w, synth.box_edge_for(w), seed=w) for w in (2500, 1100))
    fr, er, _ = oracle.forces(box.xyz, box.q, box.type, box.box, box.excl_off, box.excl_idx, synth.lj_table_spce(), rc,
                              beta, F)
    og = oracle.grid_sort(box.xyz, box.box, *shape)
    ref = oracle.pairlist(og, box.box, rl, 0.0, box.excl_off, box.excl_idx)
    ctx = mxn.nb_create(0)
    a = GpuSystem(big, shape, rl, rl, ctx=ctx)
    s = GpuSystem(box, shape, rl, rl, ctx=ctx)
    inner = mxn.nb_pairlist_prune(ctx, a.lst, a.xyzq, rl)
    other = mxn.nb_pairlist_prune(ctx, a.lst, a.xyzq, rl)
    try:
        mxn.nb_sync(ctx)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            mxn.nb_set_stream(ctx)
            mxn.nb_pairlist_prune(ctx, s.lst, s.xyzq, rl, inner)
        mxn.nb_set_stream(ctx)
        outer, s.lst = s.lst, inner
        for _ in range(4):
            graph.replay()
            mxn.nb_pairlist_prune(ctx, outer, s.xyzq, rl, other)   # eager work between the replays
            torch.cuda.synchronize()
            got = mxn.nb_list_export_canonical(inner)
            for k in ("ci", "shift", "cj", "mask"):
                np.testing.assert_array_equal(got[k], ref[k])
            f, e, _ = s.forces(rc, beta, mxn.NB_ENERGY)
            assert rel_rms(f, fr) <= 1e-5 and max_atom_err(f, fr) <= 1e-4
            np.testing.assert_allclose(e, er, rtol=1e-5)
        s.lst = outer
    finally:
        for l in (inner, other, a.lst, s.lst):
            mxn.nb_list_free(l)
        for x in (a, s):
            mxn.nb_grid_free(x.grid)
        mxn.nb_destroy(ctx)
