"""The predictor's gradient over minibatches on one workgroup, on several, and on more samples per workgroup than
it has wavefronts, against the FP64 oracle; and inside a captured graph."""
import numpy as np
import pytest

from test_gpu_buffer import HI, LO, _mlp_case

pytestmark = pytest.mark.gpu


def _grad_setup(batch):
    import torch
    import paper_1306_1737_amd as mxn
    from oracle import mlp
    p, X, y = _mlp_case(seed=batch, batch=batch)
    dev = torch.device("cuda:0")
    ctx = mxn.nb_create(0)
    m = mxn.nb_mlp_create(ctx, p, LO, HI)
    Xd, yd = torch.from_numpy(X).to(dev), torch.from_numpy(y).to(dev)
    g = torch.full((mxn.NB_MLP_PARAMS,), float("nan"), dtype=torch.float32, device=dev)
    loss = torch.zeros(1, dtype=torch.float32, device=dev)
    ref = mlp.loss_and_grad(p.astype(np.float64), mlp.normalise(X.astype(np.float64), LO, HI), y.astype(np.float64))
    return ctx, m, Xd, yd, g, loss, ref


def _check(g, loss, ref):
    # FP32 dot products of 64 terms and sums over the batch: a few 1e-7 each, 2e-5 leaves two decades
    assert float(loss.cpu()) == pytest.approx(ref[0], rel=1e-5)
    assert np.linalg.norm(g.cpu().numpy().astype(np.float64) - ref[1]) <= 2e-5 * np.linalg.norm(ref[1])


@pytest.mark.parametrize("batch", [1, 8, 9, 12, 13, 509, 513, 1031])
def test_gradient_over_batch_sizes(batch):
    import paper_1306_1737_amd as mxn
    ctx, m, Xd, yd, g, loss, ref = _grad_setup(batch)
    try:
        mxn.nb_mlp_grad(ctx, m, Xd, yd, g, loss)
        mxn.nb_sync(ctx)
        _check(g, loss, ref)
        first = g.clone()
        mxn.nb_mlp_grad(ctx, m, Xd, yd, g, loss)   # the shares are added in a fixed order
        mxn.nb_sync(ctx)
        assert (g == first).all()
        # Adam's first step moves every parameter with a clear gradient by lr against its sign
        p0 = mxn.nb_mlp_get_params(m).astype(np.float64)
        mxn.nb_mlp_train_step(ctx, m, Xd, yd, 1e-3, loss)
        p1 = mxn.nb_mlp_get_params(m).astype(np.float64)
        sel = np.abs(ref[1]) > 1e-4
        np.testing.assert_allclose((p1 - p0)[sel], -1e-3 * np.sign(ref[1][sel]), atol=2e-6)
    finally:
        mxn.nb_mlp_free(m)
        mxn.nb_destroy(ctx)


def test_gradient_in_captured_graph():
    import torch
    import paper_1306_1737_amd as mxn
    ctx, m, Xd, yd, g, loss, ref = _grad_setup(40)
    try:
        mxn.nb_sync(ctx)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            mxn.nb_set_stream(ctx)
            mxn.nb_mlp_grad(ctx, m, Xd, yd, g, loss)
        mxn.nb_set_stream(ctx)
        other = torch.zeros_like(g)
        for _ in range(3):
            g.fill_(float("nan"))
            graph.replay()
            mxn.nb_mlp_grad(ctx, m, Xd, yd, other)   # eager work between the replays
            torch.cuda.synchronize()
            _check(g, loss, ref)
            _check(other, loss, ref)
    finally:
        mxn.nb_mlp_free(m)
        mxn.nb_destroy(ctx)
