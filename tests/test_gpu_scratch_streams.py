"""The scratch of minibatches spread over workgroups on several streams and threads: each stream has rows of its own, a
stream beyond the four that have some takes them over once they lie idle, and the per-thread default stream, one handle
for a stream of every thread, gets none."""
import threading

import numpy as np
import pytest

from test_gpu_buffer import HI, LO, _mlp_case
from test_gpu_mlp_spread import _check, _grad_setup

pytestmark = pytest.mark.gpu

PER_THREAD = 2   # hipStreamPerThread


def _grads(n):
    import torch
    import paper_1306_1737_amd as mxn
    return [torch.full((mxn.NB_MLP_PARAMS,), float("nan"), dtype=torch.float32, device="cuda:0") for _ in range(n)]


def _free(ctx, m):
    import paper_1306_1737_amd as mxn
    mxn.nb_mlp_free(m)
    mxn.nb_destroy(ctx)


def test_five_streams_in_turn():
    """Calls on five streams with nothing between them that orders one after another."""
    import torch
    import paper_1306_1737_amd as mxn
    ctx, m, Xd, yd, _, _, ref = _grad_setup(509)
    try:
        streams = [torch.cuda.Stream() for _ in range(5)]
        g, losses = _grads(5), [torch.zeros(1, device="cuda:0") for _ in range(5)]
        torch.cuda.synchronize()
        for _ in range(4):
            for s, gs, ls in zip(streams, g, losses):
                mxn.nb_set_stream(ctx, s)
                mxn.nb_mlp_grad(ctx, m, Xd, yd, gs, ls)
        torch.cuda.synchronize()
        for gs, ls in zip(g, losses):
            _check(gs, ls, ref)
        for gs in g[1:4]:
            assert (gs == g[0]).all()   # the same form, rows added in a fixed order
    finally:
        _free(ctx, m)


def test_a_new_stream_takes_over_idle_rows():
    import torch
    import paper_1306_1737_amd as mxn
    ctx, m, Xd, yd, _, loss, ref = _grad_setup(256)
    try:
        streams = [torch.cuda.Stream() for _ in range(5)]
        spread, fifth = _grads(2)
        torch.cuda.synchronize()
        for s in streams[:4]:
            mxn.nb_set_stream(ctx, s)
            mxn.nb_mlp_grad(ctx, m, Xd, yd, spread, loss)
            mxn.nb_sync(ctx)
        held = mxn.nb_memory_info(ctx)
        mxn.nb_set_stream(ctx, streams[4])
        mxn.nb_mlp_grad(ctx, m, Xd, yd, fifth, loss)
        mxn.nb_sync(ctx)
        _check(fifth, loss, ref)
        assert not (fifth == spread).all()   # one workgroup: another order of the sums
        for _ in range(80):
            mxn.nb_mlp_grad(ctx, m, Xd, yd, fifth, loss)
        mxn.nb_sync(ctx)
        assert (fifth == spread).all()
        assert mxn.nb_memory_info(ctx) == held
    finally:
        _free(ctx, m)


def test_per_thread_stream_takes_no_rows():
    import torch
    import paper_1306_1737_amd as mxn
    ctx, m, Xd, yd, g, loss, ref = _grad_setup(300)
    try:
        torch.cuda.synchronize()
        held = mxn.nb_memory_info(ctx)
        mxn.nb_set_stream(ctx, PER_THREAD)
        mxn.nb_mlp_grad(ctx, m, Xd, yd, g, loss)
        mxn.nb_sync(ctx)
        _check(g, loss, ref)
        assert mxn.nb_memory_info(ctx) == held
    finally:
        _free(ctx, m)


@pytest.mark.parametrize("per_thread", [False, True])
def test_two_threads(per_thread):
    """Two threads on one model, on one stream or on their own default streams."""
    import torch
    import paper_1306_1737_amd as mxn
    ctx, m, X0, y0, _, _, ref0 = _grad_setup(509)
    try:
        from oracle import mlp
        p, X, y = _mlp_case(seed=509, batch=509)
        X, y = X[:300], y[:300]
        ref1 = mlp.loss_and_grad(p.astype(np.float64), mlp.normalise(X.astype(np.float64), LO, HI),
                                 y.astype(np.float64))
        jobs = [(X0, y0, ref0), (torch.from_numpy(X).to("cuda:0"), torch.from_numpy(y).to("cuda:0"), ref1)]
        g, losses = _grads(2), [torch.zeros(1, device="cuda:0") for _ in range(2)]
        torch.cuda.synchronize()
        if per_thread:
            mxn.nb_set_stream(ctx, PER_THREAD)
        errors = []

        def work(k):
            try:
                for _ in range(30):
                    mxn.nb_mlp_grad(ctx, m, jobs[k][0], jobs[k][1], g[k], losses[k])
                mxn.nb_sync(ctx)
            except Exception as e:
                errors.append(e)

        threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not errors, errors
        torch.cuda.synchronize()
        for k in range(2):
            _check(g[k], losses[k], jobs[k][2])
    finally:
        _free(ctx, m)
