"""Pair statistics against the oracle's pair counts, over lists with fewer and more work items than the statistics kernel
has wavefronts, with short items and with the full ones of a batch."""
import numpy as np
import pytest

import oracle
import synth
from _nb import GpuSystem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 4), (4, 8), (8, 4), (8, 8)])
@pytest.mark.parametrize("waters", [70, 300, 1500, 4500])
def test_counts(shape, waters):
    import torch
    import paper_1306_1737_amd as mxn
    rc, rl = 0.55, 0.6
    box = synth.water_box(waters, synth.box_edge_for(waters), seed=waters)
    og = oracle.grid_sort(box.xyz, box.box, *shape)
    every, kept = (int(oracle.rdf(og, og["xs"], box.type, box.box, rc, 1, 2, box.excl_off, box.excl_idx, skip).sum())
                   for skip in (False, True))
    s = GpuSystem(box, shape, rl)
    try:
        entries, items = mxn.nb_list_info(s.lst)
        got = mxn.nb_list_stats(s.ctx, s.grid, s.lst, s.xyzq, rc)
        assert got[0] == entries * shape[0] * shape[1]
        assert got[2:] == (kept, every - kept)
        # real pairs: the mask bits, and the excluded pairs that it clears (all within a water, so within rlist)
        bits = sum(bin(int(m)).count("1") for m in mxn.nb_list_export_canonical(s.lst)["mask"])
        assert got[1] == bits + 3 * waters
        f = torch.zeros((box.n, 3), dtype=torch.float32, device=s.dev)
        b = mxn.nb_batch_create(s.ctx, [s.grid], [s.lst], [s.xyzq], [f])
        assert mxn.nb_list_info(s.lst)[1] <= items
        assert mxn.nb_list_stats(s.ctx, s.grid, s.lst, s.xyzq, rc) == got
        mxn.nb_batch_free(b)
    finally:
        s.close()
