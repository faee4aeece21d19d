"""The scans that end a list build, by one workgroup and by tiles in two launches (beyond 16384 regions or j-clusters):
forces against the oracle on lists rebuilt and pruned several times (the counters start cleared every time)."""
import numpy as np
import pytest

import oracle
import synth
from _nb import F, GpuSystem, max_atom_err, rel_rms

pytestmark = pytest.mark.gpu


# 4x4: 5000 waters give about 4000 j-clusters (one tile), 20500 about 16400 of them (either side of four tiles),
# 28000 about 22000 (six tiles, the last one ragged)
@pytest.mark.parametrize("waters", [4900, 20500, 28000])
@pytest.mark.parametrize("shape", [(4, 4), (8, 4), (4, 8)])
def test_rebuilt_and_pruned(waters, shape):
    import paper_1306_1737_amd as mxn
    rc, beta = 0.6, 5.2
    box = synth.water_box(waters, synth.box_edge_for(waters), seed=waters)
    fr, er, _ = oracle.forces(box.xyz, box.q, box.type, box.box, box.excl_off, box.excl_idx, synth.lj_table_spce(), rc,
                              beta, F, mode="binned")
    s = GpuSystem(box, shape, 0.7)
    inner = None
    try:
        first = None
        for flags in (0, mxn.NB_LIST_ASYNC, mxn.NB_LIST_ASYNC, 0):
            mxn.nb_pairlist_build(s.ctx, s.grid, 0.7, -1.0, s.eo, s.ei, flags, s.lst)
            inner = mxn.nb_pairlist_prune(s.ctx, s.lst, s.xyzq, 0.7, inner)
            f, e, _ = s.forces(rc, beta, mxn.NB_ENERGY)
            if first is None:
                assert rel_rms(f, fr) <= 1e-5 and max_atom_err(f, fr) <= 1e-4
                np.testing.assert_allclose(e, er, rtol=1e-5)
                first = f
            np.testing.assert_array_equal(f, first)   # whatever order the rows got
        whole, s.lst = s.lst, inner
        f, e, _ = s.forces(rc, beta, mxn.NB_ENERGY)
        s.lst = whole
        assert rel_rms(f, fr) <= 1e-5 and max_atom_err(f, fr) <= 1e-4
        np.testing.assert_allclose(e, er, rtol=1e-5)
    finally:
        if inner is not None:
            mxn.nb_list_free(inner)
        s.close()
