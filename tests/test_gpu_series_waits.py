"""The one-launch Chebyshev series of small FP64 boxes when its workgroups cannot wait for
each other: the finishing kernel runs it alone, is counted, and gives the same bits."""
import threading

import numpy as np
import pytest
import torch

from paper_1203_6208_amd import inputs, rpy

pytestmark = pytest.mark.gpu
SIZES = [(1, 5), (10, 10), (16, 16), (1, 257), (9, 43), (32, 16), (27, 19), (24, 32), (7, 127), (32, 32)]


def _setup(size, **kw):
    w = inputs.Workload("waits", *size, 1.0, seed=93)
    return w, torch.from_numpy(w.positions()).cuda(), rpy.context_for(w, cheb_keep=140, **kw)


def _vec(w, seed=5):
    return torch.from_numpy(np.random.default_rng(seed).standard_normal((1, w.n, 3))).cuda() * 0.03


@pytest.mark.parametrize("size", [(10, 10), (20, 20), (40, 25)])
def test_count(size):
    """Series run alone are counted, others are not."""
    w, pos, a = _setup(size)
    v = _vec(w)
    bp = rpy.make_bd_params(dt=1e-3, n_cheb=20, d_min=0.04, d_max=40.0)
    a.build(pos)
    for limit, want in ((None, 0), (-1, 7), (1000000, 0)):
        if limit is not None:
            rpy.rpy_series_wait(a.handle, limit)
        p = pos.clone()
        for step in range(5):
            a.step(p, bp, seed=1, step=step)
        a.build(pos)
        a.sqrt_apply(v, 30, 0.04, 40.0)
        a.sqrt_adaptive(v, 0.04, 40.0, 1e-2, 60)
        assert rpy.rpy_series_stats(a.handle) == want
        assert rpy.rpy_series_stats(a.handle) == 0


@pytest.mark.parametrize("size", SIZES)
def test_alone_same_bits(size):
    """With every wait denied: the same bits as the series kernel, of every output, at the
    edges of its workgroups and column blocks, for fixed and adaptive orders and for steps
    of every rule."""
    w, pos, a = _setup(size)
    b = rpy.context_for(w, cheb_keep=140)
    rpy.rpy_series_wait(b.handle, -1)
    v = _vec(w)
    for c in (a, b):
        c.build(pos)
    # the product rules only where they bracket the spectrum (else the series diverges)
    hi = 1.1 * a.lanczos_bounds(min(40, 3 * w.n), margin=0.0)[1]
    for n in (2, 3, 4, 17, 65, 128):
        for x, y in zip(*(c.sqrt_apply(v, n, 0.04, 40.0, want_ef=True) for c in (a, b))):
            assert torch.equal(x, y)
        assert torch.equal(*(c.sqrt_apply(v, n, 0.04, 40.0) for c in (a, b)))
    for tol, start, nmax in ((1e-2, 0, 64), (1e-3, 2, 100), (1e-14, 3, 7), (1e-2, 0, 2), (1e-6, 30, 128)):
        x, y = (c.sqrt_adaptive(v, 0.04, 40.0, tol, nmax, n_start=start, allow_etol=True) for c in (a, b))
        assert torch.equal(x[0], y[0]) and torch.equal(x[1], y[1]) and x[2] == y[2]
    assert a.order_stats() == b.order_stats()
    assert a.status() == b.status()
    for kw in (dict(n_cheb=2, d_min=0.04, d_max=40.0), dict(n_cheb=20, d_min=0.04, d_max=40.0),
               dict(n_cheb=20, bounds_rule=rpy.BOUNDS_PAPER, bounds_C=60.0),
               dict(n_cheb=0, d_min=0.04, d_max=40.0, tol=1e-2, n_max=60),
               dict(n_cheb=0, bounds_rule=rpy.BOUNDS_PAPER, bounds_C=60.0, tol=1e-2, n_max=100)):
        if "bounds_rule" in kw and a.bounds(60.0)[1] < hi:
            continue
        bp = rpy.make_bd_params(dt=1e-3, **kw)
        p, q = pos.clone(), pos.clone()
        for step in range(3):
            x, y = (c.step(r, bp, seed=3, step=step, want=step != 1) for c, r in ((a, p), (b, q)))
            for s, t in zip(x or (), y or ()):
                assert torch.equal(s, t)
        assert torch.equal(p, q)
    assert rpy.rpy_series_stats(a.handle) == 0 and rpy.rpy_series_stats(b.handle) > 20


def test_threads_on_the_per_thread_stream():
    """Four large boxes in four threads, each on its own per-thread default stream (one handle
    value for all): their series are ordered, no wait runs out.  The threads live until the
    device is idle, since that stream ends with its thread."""
    class PerThread:
        cuda_stream = 2   # hipStreamPerThread

    n = 4
    jobs = [_setup((40, 25)) for _ in range(n)]
    v = _vec(jobs[0][0])
    outs = [torch.empty_like(v) for _ in jobs]
    for _, pos, c in jobs:
        c.build(pos)
    want = jobs[0][2].sqrt_apply(v, 128, 0.03, 40.0)
    start, idle = threading.Barrier(n + 1), threading.Event()
    enqueued = threading.Barrier(n + 1)
    torch.cuda.synchronize()

    def run(k):
        start.wait()
        for i in range(150):
            rpy.chebyshev_sqrt_apply(jobs[k][2].handle, v, outs[k], 1, 128 - (i + k) % 3, 0.03, 40.0, stream=PerThread)
        rpy.chebyshev_sqrt_apply(jobs[k][2].handle, v, outs[k], 1, 128, 0.03, 40.0, stream=PerThread)
        enqueued.wait()
        idle.wait()

    th = [threading.Thread(target=run, args=(k,)) for k in range(n)]
    for t in th:
        t.start()
    start.wait()
    enqueued.wait()
    torch.cuda.synchronize()
    idle.set()
    for t in th:
        t.join()
    for o in outs:
        assert torch.equal(o, want)
    assert [rpy.rpy_series_stats(c.handle) for _, _, c in jobs] == [0] * n


@pytest.mark.parametrize("size", [(10, 10), (32, 16), (40, 25)])
def test_numbers_start_again(size):
    """Where the terms' numbers run out of 32 bits, in every position of a call: no word of an
    earlier call, and no word never written, is taken for one of this."""
    w, pos, a = _setup(size)
    v = _vec(w)
    a.build(pos)
    want = a.sqrt_apply(v, 9, 0.04, 40.0, want_ef=True)
    ad = a.sqrt_adaptive(v, 0.04, 40.0, 1e-2, 60, n_start=2)
    for back in range(1, 16):
        # each time a new context: the words of the sums are still unwritten there
        c = rpy.context_for(w, cheb_keep=140)
        c.build(pos)
        assert torch.equal(c.sqrt_apply(v, 9, 0.04, 40.0), want[0])
        rpy._lib.rpy_series_number(c.handle, 2 ** 32 - back)
        x = c.sqrt_apply(v, 9, 0.04, 40.0, want_ef=True)
        assert torch.equal(x[0], want[0]) and torch.equal(x[1], want[1])
        rpy._lib.rpy_series_number(c.handle, 2 ** 32 - back)
        x = c.sqrt_adaptive(v, 0.04, 40.0, 1e-2, 60, n_start=2)
        assert torch.equal(x[0], ad[0]) and torch.equal(x[1], ad[1]) and x[2] == ad[2]
        assert torch.equal(c.sqrt_apply(v, 9, 0.04, 40.0), want[0])
        assert rpy.rpy_series_stats(c.handle) == 0
        c.close()
