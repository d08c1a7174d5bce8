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
