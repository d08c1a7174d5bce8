"""The reciprocal gradient's workgroups: bead counts around 64 and around the
changes of the number of parts, groups of pairs that do not fill eight, against
the oracle's reverse mode."""
import numpy as np
import pytest
import torch

import oracle
from paper_1203_6208_amd import inputs, rpy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [(1, 5), (1, 63), (13, 5), (2, 65), (1, 257), (27, 19)])
@pytest.mark.parametrize("n_cheb", [2, 9, 14])
def test_u_vjp_sizes(size, n_cheb):
    w = inputs.Workload("gedge", *size, 1.0, seed=95)
    p = w.positions()
    pos = torch.from_numpy(p).cuda()
    ctx = rpy.context_for(w, cheb_keep=16, grad=1)
    rng = np.random.default_rng(9)
    F, dw, g = (rng.standard_normal((w.n, 3)) for _ in range(3))
    gp, gF = torch.empty_like(pos), torch.empty_like(pos)
    cuda = [torch.from_numpy(a).cuda() for a in (F, dw, g)]
    rpy.rpy_u_vjp(ctx.handle, pos, *cuda, n_cheb, 0.05, 30.0, gp, gF, None)
    wp, wF = oracle.u_vjp(p, w.L, w.a, w.alpha, w.rc, w.n2max, F, dw, g, n_cheb, 0.05, 30.0)
    # as every test of the reverse mode: 1e-10 of the largest component, D g to 1e-12
    assert np.abs(gp.cpu().numpy() - wp).max() <= 1e-10 * np.abs(wp).max()
    assert np.abs(gF.cpu().numpy() - wF).max() <= 1e-12 * np.abs(wF).max()
    ctx.close()
