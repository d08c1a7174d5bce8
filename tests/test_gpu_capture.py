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
