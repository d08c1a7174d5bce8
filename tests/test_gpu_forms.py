"""Which form of D a call takes (tiles, or the complete tensor by rows): it follows from
the box, the number of vectors and the call's products alone, not from what earlier
calls formed."""
import numpy as np
import pytest
import torch

from paper_1203_6208_amd import inputs, rpy

pytestmark = pytest.mark.gpu


def _setup(size, M=3.5, **kw):
    w = inputs.Workload("forms", *size, 1.0, M=M, seed=92)
    pos = torch.from_numpy(w.positions()).cuda()
    return w, pos, rpy.context_for(w, **kw)


def _vec(w, m):
    return torch.from_numpy(np.random.default_rng(m).standard_normal((m, w.n, 3))).cuda()


@pytest.mark.parametrize("size", [(10, 10), (1, 257), (20, 20), (40, 25), (64, 18), (64, 24)])
@pytest.mark.parametrize("M", [3.5, 4.6])
def test_history_independent(size, M):
    """The same product before and after calls that form the rows: the same bits."""
    w, pos, a = _setup(size, M, max_rhs=16, cheb_keep=40)
    bp = rpy.make_bd_params(dt=1e-6, n_cheb=20, d_min=0.04, d_max=40.0)
    vs = [_vec(w, m) for m in (1, 2, 3, 4, 16)]
    a.build(pos)
    first = [a.apply(v) for v in vs]
    few = [a.sqrt_apply(v, 4, 0.04, 40.0) for v in vs]
    many = [a.sqrt_apply(v, 20, 0.04, 40.0) for v in vs]
    for call in (lambda: a.sqrt_apply(vs[0], 20, 0.04, 40.0), lambda: a.lanczos_bounds(20),
                 lambda: a.sqrt_apply(vs[2], 20, 0.04, 40.0), lambda: a.real_space_dense(),
                 lambda: a.step(pos.clone(), bp, seed=1, step=0)):
        call()
        for got, want in zip([a.apply(v) for v in vs], first):
            assert torch.equal(got, want)
        for got, want in zip([a.sqrt_apply(v, 4, 0.04, 40.0) for v in vs], few):
            assert torch.equal(got, want)
        for got, want in zip([a.sqrt_apply(v, 20, 0.04, 40.0) for v in vs], many):
            assert torch.equal(got, want)
