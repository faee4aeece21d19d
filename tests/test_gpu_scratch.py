"""Calls that take scratch when they can get it (nb_rdf over many workgroups, minibatches spread over workgroups): with
the scratch refused and HIP's error of the refusal still set, the call does its work once, in its other form, and
reports success."""
import ctypes

import numpy as np
import pytest

import synth
from _nb import GpuSystem
from test_gpu_buffer import HI, LO, _mlp_case

pytestmark = pytest.mark.gpu

BIG = 1 << 20   # the scratch of both calls is above this, every other block that they may ask for below it


class Refusing:
    """torch's allocator; while `on`, a large block is refused the way a failed hipMalloc refuses it (its error stays
    HIP's last one)."""

    def __init__(self, mxn):
        inner = mxn.torch_allocator(0)
        self.on, self.refused = False, 0

        def alloc(nbytes, stream, user):
            if self.on and nbytes >= BIG:
                p = ctypes.c_void_p()
                assert mxn.lib().hipMalloc(ctypes.byref(p), ctypes.c_size_t(1 << 60)) != 0
                self.refused += 1
                return None
            return inner.alloc(nbytes, stream, user)

        self.struct = mxn.nb_allocator(mxn._ALLOC_FN(alloc), inner.free, None)
        self._keep = inner


def test_pair_histogram():
    import torch
    import paper_1306_1737_amd as mxn
    box = synth.water_box(6000, synth.box_edge_for(6000), seed=17)
    al = Refusing(mxn)
    ctx = mxn.nb_create(0, allocator=al.struct)
    small = GpuSystem(synth.water_box(150, synth.box_edge_for(150), seed=3), (8, 8), 0.7, ctx=ctx)
    s = GpuSystem(box, (8, 8), 0.9, 0.9, ctx=ctx)
    try:
        nb, rmax = 200, 0.65
        hist = torch.zeros(4 * nb, dtype=torch.int64, device=s.dev)
        mxn.nb_rdf(ctx, small.grid, small.lst, small.xyzq, rmax, nb, 2, hist)   # uploads the edges; no scratch
        hist.zero_()
        before = mxn.nb_last_error()
        al.on = True
        mxn.nb_rdf(ctx, s.grid, s.lst, s.xyzq, rmax, nb, 2, hist)
        al.on = False
        mxn.nb_sync(ctx)
        assert al.refused == 1 and mxn.nb_last_error() == before
        refused = hist.clone()
        hist.zero_()
        mxn.nb_rdf(ctx, s.grid, s.lst, s.xyzq, rmax, nb, 2, hist)
        mxn.nb_sync(ctx)
        assert (refused == hist).all() and int(hist.sum()) > 0
    finally:
        for x in (small, s):
            mxn.nb_list_free(x.lst)
            mxn.nb_grid_free(x.grid)
        mxn.nb_destroy(ctx)


def test_training_step():
    import torch
    import paper_1306_1737_amd as mxn
    from oracle import mlp
    p, X, y = _mlp_case(seed=8, batch=64)
    al = Refusing(mxn)
    ctx = mxn.nb_create(0, allocator=al.struct)
    m = mxn.nb_mlp_create(ctx, p, LO, HI)
    try:
        dev = torch.device("cuda:0")
        Xd, yd = torch.from_numpy(X).to(dev), torch.from_numpy(y).to(dev)
        _, ref = mlp.loss_and_grad(p.astype(np.float64), mlp.normalise(X.astype(np.float64), LO, HI),
                                   y.astype(np.float64))
        al.on = True
        mxn.nb_mlp_train_step(ctx, m, Xd, yd, 1e-3)
        al.on = False
        mxn.nb_sync(ctx)
        assert al.refused == 1
        step = mxn.nb_mlp_get_params(m).astype(np.float64) - p
        sel = np.abs(ref) > 1e-4   # Adam's first step: lr against the gradient's sign
        np.testing.assert_allclose(step[sel], -1e-3 * np.sign(ref[sel]), atol=2e-6)
    finally:
        mxn.nb_mlp_free(m)
        mxn.nb_destroy(ctx)
