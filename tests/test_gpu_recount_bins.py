"""Recount histograms on the LDS path (up to 2048 bins) and beyond it, and on lists of few and many workgroups: coarse
bins add up from fine ones, and both match the oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 4), (4, 8), (8, 4), (8, 8)])
@pytest.mark.parametrize("waters", [216, 1000])
def test_histogram_sizes(shape, waters):
    import torch
    import paper_1306_1737_amd as mxn
    L = synth.box_edge_for(waters)
    box = synth.water_box(waters, L, seed=waters)
    rc, span = np.float32(0.6), 0.256
    rl = np.float32(rc + span)
    c_bb = np.float32(0.5 * (max(shape) / (box.n / L ** 3)) ** (1 / 3))
    dev = torch.device("cuda:0")
    disp = synth.gaussian_displacement(box.mass, 300.0, 0.05, seed=3)
    xt = (box.xyz.astype(np.float64) + disp).astype(np.float32)
    ctx = mxn.nb_create(0)
    try:
        up = lambda a: torch.from_numpy(a).to(dev)
        eo, ei = up(box.excl_off), up(box.excl_idx)
        lj = up(synth.lj_table_spce().astype(np.float32))
        x0, typ = up(box.xyzq()), up(box.type)
        g = mxn.nb_grid_sort(ctx, box.box, x0, typ, shape)
        lst = mxn.nb_pairlist_build(ctx, g, float(rl), float(np.float32(rl - c_bb)), eo, ei)
        p = mxn.make_params(float(rc), 5.0, synth.COULOMB_F, lj)
        got = {}
        for nbins in (1, 128, 2048, 4096):
            h = torch.full((nbins,), float("nan"), dtype=torch.float64, device=dev)
            mxn.nb_recount(ctx, g, lst, up(box.xyzq(xt)), p, float(c_bb), span / nbins, nbins, h)
            mxn.nb_sync(ctx)
            got[nbins] = h.cpu().numpy()
        # the same FP32 contributions in other bins: sums agree to FP64 rounding
        scale = np.abs(got[4096]).sum()
        assert scale > 0.0
        for nbins in (1, 128, 2048):
            assert abs(got[nbins].sum() - got[4096].sum()) <= 1e-12 * scale
        # bin widths are exact powers of two of one another: fine bins add up to the coarse ones
        np.testing.assert_allclose(got[4096].reshape(2048, 2).sum(1), got[2048], rtol=0, atol=1e-12 * scale)
        # and 128 of them match the oracle (tolerance as for the recount of a single size)
        ref = oracle.recount(box.xyz, xt, box.q, box.type, box.box, box.excl_off, box.excl_idx, synth.lj_table_spce(),
                             rc, 5.0, synth.COULOMB_F, shape[0], shape[1], rl, c_bb, span / 128, 128)
        np.testing.assert_allclose(np.cumsum(got[128][::-1])[::-1], np.cumsum(ref[::-1])[::-1], rtol=2e-3,
                                   atol=2e-4 * np.abs(ref).sum())
        mxn.nb_list_free(lst)
        mxn.nb_grid_free(g)
    finally:
        mxn.nb_destroy(ctx)
