"""The complete tensor by rows (small FP64 boxes) against the tile form: the
same calls on a context with an FP32 copy, whose FP64 products always run by
tiles, and against the oracle.  Sizes at the edges of the column blocks and of
the waves per row, both wave-vector sets, every epilogue, and the routes
between the two forms (block products, the dense copy, graph capture)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1203_6208_amd import inputs, rpy

pytestmark = pytest.mark.gpu
# both forms agree with the oracle to 1e-12; against each other the same
TOL = 1e-12


def _pair(chains, bpc, alphaL=6.0, M=3.5, **kw):
    w = inputs.Workload("rows", chains, bpc, 1.0, alphaL=alphaL, M=M, seed=77)
    pos = torch.from_numpy(w.positions()).cuda()
    return w, pos, rpy.context_for(w, **kw), rpy.context_for(w, lowp="f32", **kw)


def _vec(w, m, seed=5):
    return torch.from_numpy(np.random.default_rng(seed).standard_normal((m, w.n, 3))).cuda()


def _close(a, b, tol=TOL):
    assert torch.max(torch.abs(a - b)).item() <= tol * torch.max(torch.abs(b)).item()


SIZES = [(1, 5), (7, 9), (8, 8), (5, 13), (12, 10), (16, 16), (1, 257), (32, 16), (27, 19),
         (64, 16), (25, 41), (64, 24), (29, 53)]


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("form", [(6.0, 3.5), (6.0, 4.6), (4.0, 3.5), (8.0, 3.5)])
def test_products(size, form):
    if form != (6.0, 3.5) and size[0] * size[1] > 600:
        pytest.skip("one large size per wave-vector set is enough")
    w, pos, a, b = _pair(*size, *form, max_rhs=4)
    lo, hi = 0.05, 12.0
    for c in (a, b):
        c.build(pos)
    for m in (1, 2, 3, 4):
        v = _vec(w, m)
        _close(a.apply(v), b.apply(v))                       # tiles above the eager limit
        _close(a.sqrt_apply(v, 12, lo, hi), b.sqrt_apply(v, 12, lo, hi))
        _close(a.apply(v), b.apply(v))                       # rows: formed by the series


@pytest.mark.parametrize("size", [(10, 10), (20, 20), (25, 41)])
def test_against_oracle(size):
    w, pos, a, _ = _pair(*size)
    a.build(pos)
    v = _vec(w, 1)
    a.sqrt_apply(v, 12, 0.05, 12.0)
    D = oracle.diffusion_matrix(pos.cpu().numpy(), w.L, w.a, w.alpha, w.rc, w.n2max)
    want = (D @ v.cpu().numpy().reshape(-1)).reshape(1, -1, 3)
    _close(a.apply(v), torch.from_numpy(want).cuda())


@pytest.mark.parametrize("size", [(10, 10), (20, 20), (25, 41)])
def test_steps(size):
    """Fixed and adaptive steps under every interval rule."""
    w, pos, a, b = _pair(*size, cheb_keep=96)
    for kw in (dict(n_cheb=15, d_min=0.03, d_max=40.0),
               dict(n_cheb=15, bounds_rule=rpy.BOUNDS_PAPER, bounds_C=60.0),
               dict(n_cheb=15, bounds_rule=rpy.BOUNDS_DILUTE),
               dict(n_cheb=0, d_min=0.03, d_max=40.0, tol=1e-2, n_max=60),
               dict(n_cheb=80, d_min=0.03, d_max=40.0, tol=1e-9, n_max=84)):
        bp = rpy.make_bd_params(dt=1e-3, **kw)
        got = []
        for c in (a, b):
            p = pos.clone()
            drift, noise, ef = c.step(p, bp, seed=3, step=1, want=True)
            got.append((p, drift, noise, c.order_stats() if kw.get("tol") else None))
        for x, y in zip(got[0][:3], got[1][:3]):
            _close(x, y, 1e-11)   # the dilute interval lets T_p grow past [-1, 1]
        assert got[0][3] == got[1][3]


def test_forms_and_capture():
    """Products of 16 vectors and the dense copy form the tiles on demand, a new
    build is seen by every form, and captured calls replay on the positions of
    the replay, interleaved with eager work."""
    w, pos, a, b = _pair(12, 10, max_rhs=16)
    v1, v16 = _vec(w, 1), _vec(w, 16)
    pos2 = pos + 0.37 * _vec(w, 1, 9)[0]
    for p in (pos, pos2):
        a.build(p)
        b.build(p)
        _close(a.apply(v1), b.apply(v1))
        _close(a.apply(v16), b.apply(v16))
        _close(a.real_space_dense(), b.real_space_dense())
        _close(a.sqrt_apply(v1, 12, 0.05, 12.0), b.sqrt_apply(v1, 12, 0.05, 12.0))
    p = pos.clone()
    out = torch.empty_like(v1)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        a.build(p)
        rpy.rpy_apply(a.handle, v1, out, 1)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            a.build(p)
            rpy.rpy_apply(a.handle, v1, out, 1)
        for q in (pos2, pos, pos2):
            p.copy_(q)
            g.replay()
            s.synchronize()
            b.build(q)
            want = b.apply(v1)
            _close(out, want)
            _close(a.apply(v1), want)                 # eager, on the replay's positions
            a.build(pos)
            b.build(pos)
            _close(a.apply(v1), b.apply(v1))
            s.synchronize()


@pytest.mark.parametrize("size", [(1, 5), (10, 10), (5, 13), (16, 16), (9, 43), (64, 8)])
@pytest.mark.parametrize("alone", [False, True])
def test_series(size, alone):
    """The series kernel (every order, rule and optional output) and, with waits
    that give up at once, the finishing kernel that then runs the series alone,
    against products by tiles; calls in a row, so that a term number of an
    earlier call is never taken for one of this."""
    import ctypes
    w, pos, a, b = _pair(*size, cheb_keep=140)
    if alone:
        rpy._lib.rpy_series_wait(a.handle, ctypes.c_int64(-1))
    v = _vec(w, 1) * 0.03
    a.build(pos)
    b.build(pos)
    for n in (2, 3, 4, 17, 40, 128):
        got, want = a.sqrt_apply(v, n, 0.04, 40.0, want_ef=True), b.sqrt_apply(v, n, 0.04, 40.0, want_ef=True)
        _close(got[0], want[0])
        # E_f^2 is a difference of sums over 3N terms, rounded to about 1e-13
        assert abs(got[1].item() ** 2 - want[1].item() ** 2) < 1e-12
    for tol, start, nmax in ((1e-2, 0, 64), (1e-3, 2, 100), (1e-14, 3, 7), (1e-2, 0, 2), (1e-6, 30, 128)):
        got = a.sqrt_adaptive(v, 0.04, 40.0, tol, nmax, n_start=start, allow_etol=True)
        want = b.sqrt_adaptive(v, 0.04, 40.0, tol, nmax, n_start=start, allow_etol=True)
        assert got[2] == want[2]
        _close(got[0], want[0])
    assert a.order_stats() == b.order_stats()
    assert a.status() == b.status()
    # in a box of a few beads the paper's rule can lie below the spectrum: the
    # series then diverges (T_p grows past 1e10) and two roundings of it differ freely
    rule_holds = b.bounds(60.0)[1] > 1.1 * b.lanczos_bounds(min(40, 3 * w.n), margin=0.0)[1]
    for kw in (dict(n_cheb=2, d_min=0.04, d_max=40.0), dict(n_cheb=20, d_min=0.04, d_max=40.0),
               dict(n_cheb=20, bounds_rule=rpy.BOUNDS_PAPER, bounds_C=60.0),
               dict(n_cheb=0, d_min=0.04, d_max=40.0, tol=1e-2, n_max=60),
               dict(n_cheb=0, bounds_rule=rpy.BOUNDS_PAPER, bounds_C=60.0, tol=1e-2, n_max=100)):
        if "bounds_rule" in kw and not rule_holds:
            continue
        bp = rpy.make_bd_params(dt=1e-3, **kw)
        p, q = pos.clone(), pos.clone()
        for step in range(3):
            if step == 1:
                a.step(p, bp, seed=3, step=step)
                b.step(q, bp, seed=3, step=step)
                continue
            x, y = (c.step(r, bp, seed=3, step=step, want=True) for c, r in ((a, p), (b, q)))
            _close(x[0], y[0], 1e-11)
            _close(x[1], y[1], 1e-11)
        _close(p, q)
    assert a.order_stats()[:3] == b.order_stats()[:3]


def test_series_on_streams():
    """Four contexts stepping on four streams at once, as one after the other."""
    jobs = [_pair(n, 16)[:3] for n in (6, 12, 24, 32)]
    bp = rpy.make_bd_params(dt=1e-3, n_cheb=20, d_min=0.03, d_max=40.0)
    streams = [torch.cuda.Stream() for _ in jobs]
    res = []
    for together in (False, True):
        ps = [pos.clone() for _, pos, _ in jobs]
        torch.cuda.synchronize()
        for step in range(20):
            for (w, _, c), p, s in zip(jobs, ps, streams):
                c.step(p, bp, seed=4, step=step, stream=s)
                if not together:
                    s.synchronize()
        torch.cuda.synchronize()
        res.append(ps)
    for x, y in zip(*res):
        assert torch.equal(x, y)


@pytest.mark.parametrize("alone", [False, True])
@pytest.mark.parametrize("size", [(27, 19), (43, 15), (5, 129), (24, 32), (7, 127), (25, 41), (32, 32)])
def test_series_of_larger_boxes(size, alone):
    """As test_series, past the 512 beads of a row in one wave: the edges of the
    column blocks and of the four rows per workgroup, fixed and adaptive orders,
    steps with and without products before the series, and with the waits
    denied the finishing kernel alone."""
    import ctypes
    w, pos, a, b = _pair(*size, cheb_keep=140)
    if alone:
        rpy._lib.rpy_series_wait(a.handle, ctypes.c_int64(-1))
    v = _vec(w, 1) * 0.03
    a.build(pos)
    b.build(pos)
    for n in (2, 3, 17, 40):
        got, want = (c.sqrt_apply(v, n, 0.04, 40.0, want_ef=True) for c in (a, b))
        _close(got[0], want[0])
        assert abs(got[1].item() ** 2 - want[1].item() ** 2) < 1e-12
    for tol, nmax in ((1e-2, 64), (1e-14, 9)):
        got, want = (c.sqrt_adaptive(v, 0.04, 40.0, tol, nmax, allow_etol=True) for c in (a, b))
        assert got[2] == want[2]
        _close(got[0], want[0])
    for kw in (dict(n_cheb=20, d_min=0.04, d_max=40.0),
               dict(n_cheb=20, bounds_rule=rpy.BOUNDS_PAPER, bounds_C=60.0),
               dict(n_cheb=0, d_min=0.04, d_max=40.0, tol=1e-2, n_max=60)):
        bp = rpy.make_bd_params(dt=1e-3, **kw)
        p, q = pos.clone(), pos.clone()
        for step in range(2):
            x, y = (c.step(r, bp, seed=3, step=step, want=True) for c, r in ((a, p), (b, q)))
            _close(x[0], y[0], 1e-11)
            _close(x[1], y[1], 1e-11)
        _close(p, q)


def test_larger_series_on_streams():
    """Four contexts, three of them past 512 beads, stepping from four threads on
    four streams at once, as one after the other; one of them is destroyed and made
    anew in between."""
    import threading
    sizes = [(40, 16), (24, 16), (60, 16), (40, 25)]
    bp = rpy.make_bd_params(dt=1e-3, n_cheb=20, d_min=0.03, d_max=40.0)
    streams = [torch.cuda.Stream() for _ in sizes]
    jobs = [_pair(*z)[:3] for z in sizes]
    res = []
    for together in (False, True):
        ps = [pos.clone() for _, pos, _ in jobs]
        torch.cuda.synchronize()

        def run(k, sync):
            for step in range(20):
                jobs[k][2].step(ps[k], bp, seed=4, step=step, stream=streams[k])
                if sync:
                    streams[k].synchronize()

        if together:
            th = [threading.Thread(target=run, args=(k, False)) for k in range(len(jobs))]
            for t in th:
                t.start()
            for t in th:
                t.join()
        else:
            for k in range(len(jobs)):
                run(k, True)
        torch.cuda.synchronize()
        res.append(ps)
        w = jobs[0][0]
        jobs[0][2].close()
        jobs[0] = (w, jobs[0][1], rpy.context_for(w))
    for x, y in zip(*res):
        assert torch.equal(x, y)


@pytest.mark.parametrize("size", [(1, 255), (8, 32), (1, 257), (3, 127), (32, 16)])
def test_adaptive_series_workgroups(size):
    """Adaptive series on four rows per workgroup (two waves per row), around the
    256 beads where its register limit changes: orders and sums as by products of
    tiles, on one context after a fixed order, and four contexts on four
    streams as one after the other."""
    w, pos, a, b = _pair(*size, cheb_keep=100)
    a.build(pos)
    b.build(pos)
    v = _vec(w, 1) * 0.03
    for n, tol in ((7, 1e-2), (30, 1e-3), (2, 1e-1)):
        _close(a.sqrt_apply(v, n, 0.04, 40.0), b.sqrt_apply(v, n, 0.04, 40.0))
        x, y = (c.sqrt_adaptive(v, 0.04, 40.0, tol, 90, allow_etol=True) for c in (a, b))
        assert x[2] == y[2]
        _close(x[0], y[0])
        assert abs(x[1].item() ** 2 - y[1].item() ** 2) < 1e-12
    ctxs = [rpy.context_for(w, cheb_keep=100) for _ in range(4)]
    streams = [torch.cuda.Stream() for _ in ctxs]
    bp = rpy.make_bd_params(dt=1e-3, n_cheb=0, d_min=0.04, d_max=40.0, tol=1e-2, n_max=60)
    res = []
    for together in (False, True):
        ps = [pos.clone() for _ in ctxs]
        torch.cuda.synchronize()
        for step in range(12):
            for k, (c, s) in enumerate(zip(ctxs, streams)):
                c.step(ps[k], bp, seed=k, step=step, stream=s)
                if not together:
                    s.synchronize()
        torch.cuda.synchronize()
        res.append(ps)
    for x, y in zip(*res):
        assert torch.equal(x, y)
