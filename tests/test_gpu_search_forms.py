"""The cluster-pair search where its parts meet: boxes barely wider than 2 rlist (most image shifts populated), flat
and tall boxes, few and many grid columns, search parts, exclusion partners up to and beyond one per lane and in other
images, and columns that end in padding; lists bit-exact against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SHAPES = [(4, 4), (4, 8), (8, 4), (8, 8)]


def _check(xyz, box, shape, rlist, rbb, off, idx, parts=0):
    import torch
    import paper_1306_1737_amd as mxn
    n = len(xyz)
    xyzq = np.zeros((n, 4), np.float32)
    xyzq[:, :3] = xyz
    dev = torch.device("cuda:0")
    ctx = mxn.nb_create(0)
    try:
        mxn.nb_set_search_parts(ctx, parts)
        up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
        xq, ty, eo, ei = up(xyzq), up(np.zeros(n, np.int32)), up(off.astype(np.int32)), up(idx.astype(np.int32))
        g = mxn.nb_grid_sort(ctx, box, xq, ty, shape)
        og = oracle.grid_sort(xyz, box, *shape)
        spacing = (max(shape) / (n / np.prod(box))) ** (1 / 3)
        rb = max(0.0, rlist - 0.5 * spacing) if rbb < 0 else rbb
        ref = oracle.pairlist(og, box, rlist, rb, off.astype(np.int32), idx.astype(np.int32))
        lst = mxn.nb_pairlist_build(ctx, g, rlist, rb, eo, ei)
        for flags in (0, mxn.NB_LIST_ASYNC):
            lst = mxn.nb_pairlist_build(ctx, g, rlist, rb, eo, ei, flags, lst)
            mxn.nb_sync(ctx)
            got = mxn.nb_list_export_canonical(lst)
            for k in ("ci", "shift", "cj", "mask"):
                np.testing.assert_array_equal(got[k], ref[k])
        mxn.nb_list_free(lst)
        mxn.nb_grid_free(g)
        return len(ref)
    finally:
        mxn.nb_destroy(ctx)


def _exclusions(n, pairs):
    out = [set() for _ in range(n)]
    for a, b in pairs:
        if a != b:
            out[a].add(b)
            out[b].add(a)
    return (np.cumsum([0] + [len(s) for s in out]),
            np.array([v for s in out for v in sorted(s)] or [0], np.int32))


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("box,n,rlist", [((2.05, 2.05, 2.05), 700, 1.0), ((1.3, 4.0, 2.1), 900, 0.6),
                                         ((6.0, 6.0, 0.9), 1500, 0.4), ((0.9, 0.9, 20.0), 1300, 0.44),
                                         ((3.0, 3.0, 3.0), 37, 1.4), ((5.0, 5.0, 5.0), 5, 2.0)])
def test_boxes(shape, box, n, rlist):
    rng = np.random.default_rng(n)
    box = np.array(box)
    xyz = (rng.uniform(-1.0, 2.0, (n, 3)) * box).astype(np.float32)   # several images
    near = [(a, a + d) for a in range(0, n - 2, 3) for d in (1, 2)]
    off, idx = _exclusions(n, near)
    for rbb in (-1.0, 0.0, rlist):
        _check(xyz, box, shape, rlist, rbb, off, idx)


@pytest.mark.parametrize("shape", [(4, 8), (8, 8)])
@pytest.mark.parametrize("parts", [1, 2, 8])
@pytest.mark.parametrize("per", [0, 1, 7, 8, 9, 40])
def test_partners(shape, parts, per):
    """per: exclusion partners a particle gets at least, its nearest neighbours (8 x 8 = 64 fill the lanes)."""
    rng = np.random.default_rng(100 + per)
    n, box = 420, np.array([1.9, 1.7, 2.3])
    xyz = (rng.uniform(0.0, 1.0, (n, 3)) * box).astype(np.float32)
    d = xyz[:, None, :].astype(np.float64) - xyz[None]
    d -= np.round(d / box) * box
    order = np.argsort((d ** 2).sum(-1), axis=1)
    off, idx = _exclusions(n, [(a, int(b)) for a in range(n) for b in order[a, 1:per + 1]])
    assert _check(xyz, box, shape, 0.8, -1.0, off, idx, parts) > 0
