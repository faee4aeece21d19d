"""Particles many boxes away, whose image shift k L is not a float: the positions that the force, histogram and prune calls
gather are the sort's own, so histograms are the oracle's count for count and a list pruned at its build positions is the
one-stage list."""
import numpy as np
import pytest

import oracle
from _nb import rel_rms

pytestmark = pytest.mark.gpu

SHAPES = [(4, 4), (4, 8), (8, 4), (8, 8)]


def _far(n, box, images, seed):
    rng = np.random.default_rng(seed)
    k = rng.integers(-images, images + 1, (n, 3))
    return ((rng.uniform(0.02, 0.98, (n, 3)) + k) * box).astype(np.float32)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("images", [2, 5, 100, 500])
def test_histogram_and_prune(shape, images):
    import torch
    import paper_1306_1737_amd as mxn
    n, box, rlist, bins = 1200, np.array([3.1701, 2.9033, 2.6177]), 1.1, 900
    x = _far(n, box, images, images)
    og = oracle.grid_sort(x, box, *shape)
    off, idx = np.zeros(n + 1, np.int32), np.zeros(1, np.int32)
    xyzq = np.zeros((n, 4), np.float32)
    xyzq[:, :3] = x
    up = lambda a: torch.from_numpy(a).to("cuda:0")
    ctx = mxn.nb_create(0)
    try:
        xd, td, eo, ei = up(xyzq), up(np.zeros(n, np.int32)), up(off), up(idx)
        g = mxn.nb_grid_sort(ctx, box, xd, td, shape)
        outer = mxn.nb_pairlist_build(ctx, g, rlist, rlist, eo, ei)
        inner = mxn.nb_pairlist_prune(ctx, outer, xd, rlist)
        hist = torch.zeros(bins, dtype=torch.int64, device="cuda:0")
        mxn.nb_rdf(ctx, g, outer, xd, 1.0, bins, 1, hist)
        mxn.nb_sync(ctx)
        ref = oracle.rdf(og, og["xs"], np.zeros(n, np.int32), box, 1.0, bins, 1, off, idx, False)
        np.testing.assert_array_equal(hist.cpu().numpy().astype(np.uint64).reshape(1, 1, bins), ref)
        got, want = mxn.nb_list_export_canonical(inner), oracle.pairlist(og, box, rlist, 0.0, off, idx)
        for k in ("ci", "shift", "cj", "mask"):
            np.testing.assert_array_equal(got[k], want[k])
        for l in (inner, outer):
            mxn.nb_list_free(l)
        mxn.nb_grid_free(g)
    finally:
        mxn.nb_destroy(ctx)


@pytest.mark.parametrize("n", [1200, 18000])   # read through the permutation, and gathered
def test_forces(n):
    """Forces of single calls and of a batch on far images equal those of the same particles at the sort's positions."""
    import torch
    import paper_1306_1737_amd as mxn
    box = np.array([3.1701, 2.9033, 2.6177]) * (n / 1200) ** (1 / 3)
    x = _far(n, box, 400, 3)
    og = oracle.grid_sort(x, box, 8, 8)
    xyzq = np.zeros((n, 4), np.float32)
    xyzq[:, 3] = np.random.default_rng(1).normal(0.0, 1.0, n)
    ctx = mxn.nb_create(0)
    up = lambda a: torch.from_numpy(a).to("cuda:0")
    try:
        lj, td, eo, ei = (up(a) for a in (np.zeros((1, 1, 2), np.float32), np.zeros(n, np.int32), np.zeros(n + 1, np.int32),
                                          np.zeros(1, np.int32)))
        p = mxn.make_params(0.9, 3.4, 1.0, lj)
        out = []
        for pos in (x, og["xw"]):
            xyzq[:, :3] = pos
            xd = up(xyzq.copy())
            g = mxn.nb_grid_sort(ctx, box, xd, td, (8, 8))
            l = mxn.nb_pairlist_build(ctx, g, 1.0, -1.0, eo, ei)
            f = [torch.zeros((n, 3), device="cuda:0") for _ in range(2)]
            mxn.nb_forces(ctx, g, l, xd, p, 0, f[0])
            b = mxn.nb_batch_create(ctx, [g], [l], [xd], [f[1]])
            mxn.nb_batch_forces(ctx, b, p, 0)
            mxn.nb_sync(ctx)
            out.append([t.cpu().numpy() for t in f])
            mxn.nb_batch_free(b)
            mxn.nb_list_free(l)
            mxn.nb_grid_free(g)
        for far, near in zip(*out):   # the same particles, lists and order of sums
            np.testing.assert_array_equal(far, near)
        assert rel_rms(out[0][1].astype(np.float64), out[0][0].astype(np.float64)) <= 1e-6
    finally:
        mxn.nb_destroy(ctx)
