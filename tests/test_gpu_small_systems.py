"""Force calls of systems with and without a gather launch (either side of 16384 slots): forces, energies and virial
against the oracle and, bit for bit, against the FP32-accumulating call, which always gathers; positions outside the
box, all Coulomb forms; bad coordinates and types are still reported."""
import numpy as np
import pytest

import oracle
import synth
from _nb import F, max_atom_err, rel_rms

pytestmark = pytest.mark.gpu


def _system(waters, shape, rc, seed):
    import torch
    import paper_1306_1737_amd as mxn
    box = synth.water_box(waters, synth.box_edge_for(waters), seed=seed)
    rng = np.random.default_rng(seed)
    x0 = (box.xyz + rng.integers(-2, 3, box.xyz.shape) * box.box.astype(np.float32)).astype(np.float32)   # images
    dev = torch.device("cuda:0")
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ctx = mxn.nb_create(0)
    typ, eo, ei = up(box.type), up(box.excl_off), up(box.excl_idx)
    g = mxn.nb_grid_sort(ctx, box.box, up(box.xyzq(x0)), typ, shape)
    lst = mxn.nb_pairlist_build(ctx, g, rc + 0.1, -1.0, eo, ei)
    v = synth.velocities(box.mass, 300.0, seed=seed)
    xt = (x0.astype(np.float64) + v * 0.008).astype(np.float32)
    # the slot positions' definition: image moves rounded in FP32, in the build-time image
    og = oracle.grid_sort(x0, box.box, *shape)
    xref = oracle.gather(og, xt, box.box)[og["slot_of"]]
    return mxn, torch, box, ctx, g, lst, up, xt, xref


def _call(mxn, torch, box, ctx, g, lst, xq, p, flags):
    f = torch.zeros((box.n, 3), dtype=torch.float32, device=xq.device)
    e = torch.zeros(2, dtype=torch.float64, device=xq.device)
    v = torch.zeros(9, dtype=torch.float64, device=xq.device)
    mxn.nb_forces(ctx, g, lst, xq, p, flags, f, e, v)
    mxn.nb_sync(ctx)
    return f.cpu().numpy(), e.cpu().numpy(), v.cpu().numpy()


# 8x8: 96 atoms; 16384 slots lie between about 4950 and 5150 waters for every shape
@pytest.mark.parametrize("waters", [32, 1500, 5300])
@pytest.mark.parametrize("shape", [(4, 4), (4, 8), (8, 4), (8, 8)])
def test_small_and_gathered(waters, shape):
    rc = 0.35 if waters < 100 else 0.7
    mxn, torch, box, ctx, g, lst, up, xt, xref = _system(waters, shape, rc, seed=waters)
    try:
        xq = up(box.xyzq(xt))
        lj = up(synth.lj_table_spce().astype(np.float32))
        for coulomb, eps in ((mxn.NB_COULOMB_EWALD, 0.0), (mxn.NB_COULOMB_RF, 0.0), (mxn.NB_COULOMB_EWALD_TABLE, 0.0)):
            p = mxn.make_params(rc, 3.2 / rc, F, lj, coulomb=coulomb, eps_rf=eps)
            both = mxn.NB_ENERGY | mxn.NB_VIRIAL
            f0, _, _ = _call(mxn, torch, box, ctx, g, lst, xq, p, 0)
            f1, e1, v1 = _call(mxn, torch, box, ctx, g, lst, xq, p, both)
            f2, e2, _ = _call(mxn, torch, box, ctx, g, lst, xq, p, mxn.NB_ENERGY)
            f3, e3, v3 = _call(mxn, torch, box, ctx, g, lst, xq, p, both | mxn.NB_ACC_FP32)
            np.testing.assert_array_equal(f1, f3)   # the same i-force sums with the virial
            np.testing.assert_array_equal(f0, f2)
            assert rel_rms(f0.astype(np.float64), f1.astype(np.float64)) <= 2e-6
            np.testing.assert_allclose(e1, e2, rtol=1e-12)
            np.testing.assert_allclose(e1, e3, rtol=1e-5)
            np.testing.assert_allclose(v1, v3, atol=1e-5 * np.abs(v1).max())
            if coulomb == mxn.NB_COULOMB_EWALD:
                fr, er, vr = oracle.forces(xref, box.q, box.type, box.box, box.excl_off, box.excl_idx,
                                           synth.lj_table_spce(), rc, 3.2 / rc, F, mode="brute")
                assert rel_rms(f1.astype(np.float64), fr) <= 1e-5 and max_atom_err(f1.astype(np.float64), fr) <= 1e-4
                np.testing.assert_allclose(e1, er, rtol=1e-5, atol=1e-5 * np.abs(er).max())
                assert np.abs(v1.reshape(3, 3) - vr).max() <= 1e-5 * np.abs(vr).max()
    finally:
        mxn.nb_list_free(lst)
        mxn.nb_grid_free(g)
        mxn.nb_destroy(ctx)


@pytest.mark.parametrize("bad", ["nan", "type"])
def test_bad_input_reported(bad):
    mxn, torch, box, ctx, g, lst, up, xt, xref = _system(200, (8, 8), 0.7, seed=9)
    try:
        x = box.xyzq(xt)
        lj = synth.lj_table_spce().astype(np.float32)
        if bad == "nan":
            x[17, 1] = np.nan
        else:
            lj = lj[:1, :1]   # one type: the hydrogens' lies outside
        f = torch.zeros((box.n, 3), dtype=torch.float32, device="cuda:0")
        mxn.nb_forces(ctx, g, lst, up(x), mxn.make_params(0.7, 4.0, F, up(lj)), 0, f)
        with pytest.raises(mxn.NbError) as e:
            mxn.nb_sync(ctx)
        assert e.value.status == (mxn.NB_ERR_NONFINITE if bad == "nan" else mxn.NB_ERR_ARG)
    finally:
        mxn.nb_list_free(lst)
        mxn.nb_grid_free(g)
        mxn.nb_destroy(ctx)
