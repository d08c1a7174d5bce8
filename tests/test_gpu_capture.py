"""Captured calls: what a replay computes is D of the positions of the replay or of
the last build before it, whatever eager calls ran in between, and eager calls after
a replay see its positions.  Every replay is checked against an eager context."""
import numpy as np
import pytest
import torch

from paper_1203_6208_amd import inputs, rpy

pytestmark = pytest.mark.gpu
TOL = 1e-12   # two forms of D, as every FP64 product test


def _setup(size, **kw):
    w = inputs.Workload("capture", *size, 1.0, seed=91)
    p = w.positions()
    rng = np.random.default_rng(4)
    pos = [torch.from_numpy(p + 0.4 * k * rng.standard_normal(p.shape)).cuda() for k in range(3)]
    vec = {m: torch.from_numpy(rng.standard_normal((m, w.n, 3))).cuda() for m in (1, 3, 16)}
    return w, pos, vec, rpy.context_for(w, **kw), rpy.context_for(w, **kw)


def _close(a, b, tol=TOL):
    assert torch.max(torch.abs(a - b)).item() <= tol * torch.max(torch.abs(b)).item()


def _capture(s, fn):
    g = torch.cuda.CUDAGraph()
    s.synchronize()
    with torch.cuda.graph(g, stream=s):
        fn()
    return g


@pytest.mark.parametrize("size", [(10, 10), (21, 100)])
def test_block_products(size):
    """16 vectors: the phases of the structure factors belong to the positions.  A
    captured product alone follows the eager builds around it, a captured build with
    its product does not leave later eager products on older phases."""
    w, pos, vec, a, ref = _setup(size, max_rhs=16)
    v, out, out2 = vec[16], torch.empty_like(vec[16]), torch.empty_like(vec[16])
    p = pos[0].clone()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        a.build(pos[0])
        rpy.rpy_apply(a.handle, v, out, 16)
        product = _capture(s, lambda: rpy.rpy_apply(a.handle, v, out, 16))
        both = _capture(s, lambda: (a.build(p), rpy.rpy_apply(a.handle, v, out2, 16)))
        for k in (1, 2, 0, 1):
            ref.build(pos[k])
            want = ref.apply(v)
            a.build(pos[k])
            product.replay()
            _close(out, want)
            _close(a.apply(v), want)
            p.copy_(pos[(k + 1) % 3])
            both.replay()
            ref.build(p)
            want = ref.apply(v)
            _close(out2, want)
            _close(a.apply(v), want)   # eager, on the replay's positions
            product.replay()
            _close(out, want)
        s.synchronize()


def _kernels(g):
    """Kernel nodes of a captured graph."""
    import ctypes
    hip = ctypes.CDLL("libamdhip64.so")
    n = ctypes.c_size_t()
    raw = ctypes.c_void_p(g.raw_cuda_graph())
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("size", [(10, 10), (16, 16), (1, 257), (40, 16), (40, 25), (21, 100)])
def test_one_build_per_graph(size):
    """A graph of a build and products holds one build, a graph of products on a tensor
    formed before none."""
    w, pos, vec, a, _ = _setup(size)
    v, out = vec[1], torch.empty_like(vec[1])
    s = torch.cuda.Stream()

    def nodes(build, products):
        g = torch.cuda.CUDAGraph(keep_graph=True)
        s.synchronize()
        with torch.cuda.graph(g, stream=s):
            if build:
                a.build(pos[0])
            for _ in range(products):
                rpy.rpy_apply(a.handle, v, out, 1)
        return _kernels(g)

    with torch.cuda.stream(s):
        a.build(pos[0])
        rpy.rpy_apply(a.handle, v, out, 1)
        one, four = nodes(False, 1), nodes(False, 4)
        assert one <= 2 and four == 4 * one
        assert nodes(True, 4) - nodes(True, 1) == 3 * one
        assert nodes(True, 1) == one + 2   # tables, tiles or rows
        s.synchronize()


@pytest.mark.parametrize("size", [(10, 10), (16, 16), (20, 20), (40, 25), (25, 45)])
def test_replays_between_eager_calls(size):
    """Steps, builds and products captured and eager, in turn, on one context, each
    against a context that never captures: products of every form, the square root, the
    dense copy.  Eager calls give the same bits whether or not some call was captured."""
    w, pos, vec, a, ref = _setup(size, max_rhs=16, cheb_keep=64)
    v1, v3, v16 = vec[1], vec[3], vec[16]
    o1, o3, o16 = (torch.empty_like(v) for v in (v1, v3, v16))
    bp = rpy.make_bd_params(dt=1e-3, n_cheb=20, d_min=0.03, d_max=40.0)
    ap = rpy.make_bd_params(dt=1e-3, n_cheb=0, d_min=0.03, d_max=40.0, tol=1e-2, n_max=60)
    s = torch.cuda.Stream()
    p = pos[0].clone()

    def products():
        rpy.rpy_apply(a.handle, v1, o1, 1)
        rpy.rpy_apply(a.handle, v3, o3, 3)
        rpy.rpy_apply(a.handle, v16, o16, 16)

    def check_replayed():
        _close(o1, ref.apply(v1))
        _close(o3, ref.apply(v3))
        _close(o16, ref.apply(v16))

    def check_eager(same):
        for x, y in ((a.apply(v1), ref.apply(v1)), (a.apply(v3), ref.apply(v3)),
                     (a.apply(v16), ref.apply(v16)), (a.real_space_dense(), ref.real_space_dense()),
                     (a.sqrt_apply(v1, 20, 0.03, 40.0), ref.sqrt_apply(v1, 20, 0.03, 40.0)),
                     (a.sqrt_apply(v3, 20, 0.03, 40.0), ref.sqrt_apply(v3, 20, 0.03, 40.0)),
                     (a.apply(v1), ref.apply(v1))):
            assert torch.equal(x, y) if same else _close(x, y) is None

    with torch.cuda.stream(s):
        a.build(pos[0])
        products()
        g_products = _capture(s, products)
        g_build = _capture(s, lambda: a.build(p))
        g_both = _capture(s, lambda: (a.build(p), products()))
        g_step = _capture(s, lambda: a.step(p, bp, seed=5, step=1))
        g_adaptive = _capture(s, lambda: a.step(p, ap, seed=5, step=2))
        for k in (1, 2, 0, 1):
            a.build(pos[k])                       # eager build, captured products
            ref.build(pos[k])
            g_products.replay()
            check_replayed()
            check_eager(True)
            p.copy_(pos[(k + 1) % 3])             # captured build, captured and eager products
            ref.build(p)
            g_build.replay()
            g_products.replay()
            check_replayed()
            check_eager(True)
            p.copy_(pos[(k + 2) % 3])
            ref.build(p)
            g_both.replay()
            check_replayed()
            check_eager(True)
            for g, b in ((g_step, bp), (g_adaptive, ap)):
                p.copy_(pos[k])                   # captured steps; D is of their start
                q = pos[k].clone()
                g.replay()
                ref.step(q, b, seed=5, step=1 if b is bp else 2)
                _close(p, q)
                check_eager(True)
                g_products.replay()
                check_replayed()
            p.copy_(pos[k])                       # eager steps: the same bits
            q = pos[k].clone()
            for step in range(2):
                a.step(p, bp, seed=6, step=step)
                ref.step(q, bp, seed=6, step=step)
                g_products.replay()               # of an eager step's tensor
                check_replayed()
                a.step(p, ap, seed=6, step=step)
                ref.step(q, ap, seed=6, step=step)
                assert torch.equal(p, q)
        s.synchronize()
