"""Histogram bins at their edges: pairs placed exactly on, just below and just above squared bin edges, few and many
bins, three types, and distances down to zero; bit-exact against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 4), (8, 8)])
@pytest.mark.parametrize("nbins,r_max", [(1, 0.8), (7, 0.7), (100, 1.0), (1600, 0.9)])
def test_bins_at_edges(shape, nbins, r_max):
    import torch
    import paper_1306_1737_amd as mxn
    rng = np.random.default_rng(nbins)
    L, nt, m = 4.0, 3, 40
    xyz = []
    for k in range(m):   # isolated groups along a line: one centre and partners at chosen distances in x
        c = np.array([0.25 + 0.5 * (k % 8), 0.3 + 0.7 * (k // 8), 2.0], np.float32)
        xyz.append(c)
        e = rng.integers(0, nbins + 1)
        r = np.float32(e * (r_max / nbins))
        xyz += [c + np.float32([0, 0, d]) for d in (r, np.nextafter(r, np.float32(0)), np.nextafter(r, np.float32(9)))]
    xyz.append(xyz[0].copy())   # an overlapping pair
    xyz = np.array(xyz, np.float32)
    n = len(xyz)
    xyzq = np.zeros((n, 4), np.float32)
    xyzq[:, :3] = xyz
    typ = rng.integers(0, nt, n).astype(np.int32)
    box = np.array([L, L, L])
    off = np.zeros(n + 1, np.int32)
    dev = torch.device("cuda:0")
    ctx = mxn.nb_create(0)
    try:
        xq, ty, eo = (torch.from_numpy(a).to(dev) for a in (xyzq, typ, off))
        ei = torch.zeros(0, dtype=torch.int32, device=dev)
        g = mxn.nb_grid_sort(ctx, box, xq, ty, shape)
        lst = mxn.nb_pairlist_build(ctx, g, r_max + 0.01, r_max + 0.01, eo, ei)
        hist = torch.zeros(nt * nt * nbins, dtype=torch.int64, device=dev)
        mxn.nb_rdf(ctx, g, lst, xq, r_max, nbins, nt, hist)
        mxn.nb_sync(ctx)
        og = oracle.grid_sort(xyz, box, *shape)
        ref = oracle.rdf(og, og["xs"], typ, box, r_max, nbins, nt, off, np.zeros(0, np.int32), False)
        np.testing.assert_array_equal(hist.cpu().numpy().astype(np.uint64).reshape(nt, nt, nbins), ref)
        assert int(ref.sum()) > m
        mxn.nb_list_free(lst)
        mxn.nb_grid_free(g)
    finally:
        mxn.nb_destroy(ctx)


def test_many_workgroups_and_capture():
    """A box large enough for the summing launch, and the same call captured (which flushes directly)."""
    import torch
    import synth
    import paper_1306_1737_amd as mxn
    box = synth.water_box(12000, synth.box_edge_for(12000), seed=5)
    dev = torch.device("cuda:0")
    ctx = mxn.nb_create(0)
    try:
        xq, ty = torch.from_numpy(box.xyzq()).to(dev), torch.from_numpy(box.type).to(dev)
        eo, ei = torch.from_numpy(box.excl_off).to(dev), torch.from_numpy(box.excl_idx).to(dev)
        g = mxn.nb_grid_sort(ctx, box.box, xq, ty, (8, 8))
        lst = mxn.nb_pairlist_build(ctx, g, 1.01, 1.01, eo, ei)
        hist = torch.zeros(4 * 300, dtype=torch.int64, device=dev)
        mxn.nb_rdf(ctx, g, lst, xq, 1.0, 300, 2, hist)
        mxn.nb_sync(ctx)
        once = hist.clone()
        # every pair below r_max, as the list's own statistics count them
        assert int(once.sum()) == sum(mxn.nb_list_stats(ctx, g, lst, xq, 1.0)[2:])
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            mxn.nb_set_stream(ctx)
            mxn.nb_rdf(ctx, g, lst, xq, 1.0, 300, 2, hist)
        mxn.nb_set_stream(ctx)
        for k in range(3):
            graph.replay()
            mxn.nb_rdf(ctx, g, lst, xq, 1.0, 300, 2, hist)   # eager work between the replays
            torch.cuda.synchronize()
            assert (hist == (2 * k + 3) * once).all()
        mxn.nb_list_free(lst)
        mxn.nb_grid_free(g)
    finally:
        mxn.nb_destroy(ctx)
