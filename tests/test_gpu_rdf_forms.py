"""The histogram's two ways of adding its workgroups' counts, on either side of the rule that chooses between them:
counts bit-exact against the oracle with few and many counters over few and many workgroups."""
import numpy as np
import pytest

import oracle
import synth
from _nb import GpuSystem

pytestmark = pytest.mark.gpu


# counters: 4 bins; workgroups times (42 ns - 2.7 ps counters) above or below 5 us
@pytest.mark.parametrize("shape", [(4, 4), (8, 8)])
@pytest.mark.parametrize("waters,bins", [(300, 40), (300, 3000), (900, 100), (900, 3200)])
@pytest.mark.parametrize("skip", [False, True])
def test_counts(shape, waters, bins, skip):
    import torch
    import paper_1306_1737_amd as mxn
    rmax = 0.8
    box = synth.water_box(waters, synth.box_edge_for(waters), seed=waters)
    og = oracle.grid_sort(box.xyz, box.box, *shape)
    ref = oracle.rdf(og, og["xs"], box.type, box.box, rmax, bins, 2, box.excl_off, box.excl_idx, skip)
    s = GpuSystem(box, shape, 0.85, 0.85)
    try:
        hist = torch.zeros(4 * bins, dtype=torch.int64, device=s.dev)
        for k in range(1, 3):   # added to
            mxn.nb_rdf(s.ctx, s.grid, s.lst, s.xyzq, rmax, bins, 2, hist, skip)
            mxn.nb_sync(s.ctx)
            np.testing.assert_array_equal(hist.cpu().numpy().astype(np.uint64).reshape(2, 2, bins), k * ref)
    finally:
        s.close()
