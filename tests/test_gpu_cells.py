"""The cell list by one workgroup (at most 32768 beads in 4096 cells) and by
launches of their own: excluded-volume forces and low-memory products at bead
and cell counts on both sides, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1203_6208_amd import inputs, rpy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [(1, 5), (3, 341), (25, 41), (64, 33), (64, 64), (17, 241)])
@pytest.mark.parametrize("nc", [3, 10, 16, 17])
def test_ev_forces(size, nc):
    """nc cells per axis (16^3 = 4096 is the largest list of one workgroup)."""
    w = inputs.Workload("cells", *size, 1.0, seed=58)
    p = w.positions()
    pos = torch.from_numpy(p).cuda()
    rcut = w.L / (nc + 0.25)
    dstar = rcut / 8.0
    ctx = rpy.context_for(w)
    F = rpy.rpy_forces(ctx.handle, pos, 1.0, dstar, rcut, torch.empty_like(pos)).cpu().numpy()
    want = oracle.spring_forces(p, w.nchains, w.bpc) + oracle.ev_forces(p, w.L, 1.0, dstar, rcut)
    assert np.abs(F - want).max() <= 1e-12 * np.abs(want).max()   # as every FP64 force test
    again = rpy.rpy_forces(ctx.handle, pos, 1.0, dstar, rcut, torch.empty_like(pos)).cpu().numpy()
    assert np.array_equal(F, again)
    ctx.close()
