"""The real-space tiles formed from the smooth part's polynomials against the
oracle: every variant of the build (30 and 38 terms, one or several image
components moved), the parameters outside its range (which take the erfc
form), tile remainders and coincident beads, single box and batch.

Tolerance: an entry is a handful of FP64 roundings of terms of order one
(the polynomial's own error is below 2e-17), far below 1e-13 of the largest
entry, which also covers the oracle's rounding."""
import numpy as np
import pytest
import torch

import oracle
from paper_1203_6208_amd import inputs, rpy

pytestmark = pytest.mark.gpu
TOL = 1e-13

# (alpha L, M): reach over L and terms -- 0.58 / 30, 0.77 / 38, 0.875 / 30,
# 0.575 / 38; then the erfc form: a longer series, 2a > r_c
FORMS = [(6.0, 3.5), (6.0, 4.6), (4.0, 3.5), (8.0, 4.6), (6.0, 5.6), (16.0, 1.9)]


def _box(chains, bpc, alphaL, M, seed):
    w = inputs.Workload("pairs", chains, bpc, 1.0, alphaL=alphaL, M=M, seed=seed)
    pos = w.positions()
    pos[1] = pos[0]                                   # coincident
    pos[2] = pos[0] + [2.0 * w.a * (1.0 - 1e-9), 0.0, 0.0]   # at contact
    pos[3] = pos[0] + [0.5 * w.L, 0.5 * w.L, 0.0]     # on the half-box faces
    pos[4] = [0.0, 0.0, w.L]
    return w, pos


def _want(w, pos):
    return oracle.real_space_matrix(pos, w.L, w.a, w.alpha, w.rc)


@pytest.mark.parametrize("n", [(10, 10), (8, 8), (13, 5), (10, 19)])
@pytest.mark.parametrize("form", FORMS)
def test_stored_matrix(n, form):
    w, pos = _box(*n, *form, seed=41)
    with_f32 = n == (13, 5)
    ctx = rpy.context_for(w, lowp="f32" if with_f32 else "f64")
    ctx.build(torch.from_numpy(pos).cuda())
    got = ctx.real_space_dense().cpu().numpy()
    want = _want(w, pos)
    assert np.max(np.abs(got - want)) <= TOL * np.max(np.abs(want))


@pytest.mark.parametrize("tile", [32, 64])
@pytest.mark.parametrize("form", FORMS)
def test_batch_product(tile, form):
    boxes = [_box(9, 10, *form, seed=51), _box(5, 25, *form, seed=52), _box(2, 32, *form, seed=53)]
    ws = [w for w, _ in boxes]
    B = rpy.Batch(ws, tile_beads=tile)
    B.build(B.pack([p for _, p in boxes]))
    vs = [np.random.default_rng(i).standard_normal((w.n, 3)) for i, w in enumerate(ws)]
    got = B.unpack(B.apply(B.pack(vs)))
    for (w, pos), v, g in zip(boxes, vs, got):
        D = oracle.diffusion_matrix(pos, w.L, w.a, w.alpha, w.rc, w.n2max)
        want = (D @ v.reshape(-1)).reshape(-1, 3)
        # the products of this suite agree with the oracle to 1e-12
        assert np.max(np.abs(g[0].cpu().numpy() - want)) <= 1e-12 * np.max(np.abs(want))
