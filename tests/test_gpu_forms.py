"""Which form of D a call takes (tiles, or the complete tensor by rows): it follows from
the box, the number of vectors and the call's products alone, not from what earlier
calls formed."""
import numpy as np
import pytest
import torch

import oracle
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


def _by_rows(ctx, call):
    """Whether the call's products ended in no back-projection kernel."""
    rpy.rpy_profile_enable(ctx.handle, 64)
    call()
    n, _ = rpy.rpy_profile_read(ctx.handle, rpy.PROF_EPI)
    rpy.rpy_profile_enable(ctx.handle, 0)
    return n == 0


@pytest.mark.parametrize("size,M,few,many", [((16, 16), 3.5, True, True), ((1, 257), 3.5, False, True),
                                             ((32, 32), 3.5, False, True), ((32, 32), 4.6, False, True),
                                             ((25, 41), 3.5, False, False), ((25, 41), 4.6, False, True),
                                             ((64, 20), 4.6, False, True), ((21, 61), 4.6, False, False),
                                             ((64, 24), 3.5, False, False), ((64, 24), 4.6, False, False)])
def test_rule(size, M, few, many):
    """Rows for 1 to 4 vectors where they are the faster form: up to 1024 beads from 8
    products on (to 256 from the first), past it only with more than 1024 wave vectors, to
    1280 beads and from 16 products on."""
    w, pos, a = _setup(size, M, max_rhs=4)
    a.build(pos)
    for m in (1, 2, 3, 4):
        v = _vec(w, m)
        assert _by_rows(a, lambda: a.apply(v)) == few
        assert _by_rows(a, lambda: a.sqrt_apply(v, 8, 0.04, 40.0)) == few   # 7 products
        if w.n <= 1024:
            assert _by_rows(a, lambda: a.sqrt_apply(v, 9, 0.04, 40.0)) == many
        else:
            assert not _by_rows(a, lambda: a.sqrt_apply(v, 16, 0.04, 40.0))
        assert _by_rows(a, lambda: a.sqrt_apply(v, 17, 0.04, 40.0)) == many


@pytest.mark.parametrize("size,M", [((1, 257), 3.5), ((24, 32), 3.5), ((7, 127), 4.6), ((40, 25), 3.5), ((32, 32), 4.6),
                                    ((25, 41), 4.6), ((64, 18), 4.6), ((1, 1153), 4.6), ((64, 20), 4.6)])
def test_several_vectors_by_rows(size, M):
    """1 to 4 vectors per product in one launch, at the edges of the column blocks and of the
    waves per row, against the tiles of a context with an FP32 copy: Lanczos
    coefficients, fixed and adaptive square roots, steps of every interval rule."""
    w, pos, a = _setup(size, M, max_rhs=4, cheb_keep=60)
    b = rpy.context_for(w, lowp="f32", max_rhs=4, cheb_keep=60)
    a.build(pos)
    b.build(pos)
    x, y = a.lanczos_bounds(20), b.lanczos_bounds(20)
    assert np.allclose(x[2], y[2], rtol=1e-10) and np.allclose(x[3], y[3], rtol=1e-10)
    for m in (1, 2, 3, 4):
        v = _vec(w, m) * 0.03
        for p, q in ((a.sqrt_apply(v, 20, 0.04, 40.0, want_ef=True), b.sqrt_apply(v, 20, 0.04, 40.0, want_ef=True)),
                     (a.sqrt_adaptive(v, 0.04, 40.0, 1e-2, 50, allow_etol=True),
                      b.sqrt_adaptive(v, 0.04, 40.0, 1e-2, 50, allow_etol=True))):
            assert torch.max(torch.abs(p[0] - q[0])).item() <= 1e-12 * torch.max(torch.abs(q[0])).item()
            # E_f^2 is a difference of sums over 3N terms, rounded to about 1e-13
            assert torch.max(torch.abs(p[1] ** 2 - q[1] ** 2)).item() < 1e-12
            assert p[2:] == q[2:]
    for kw in (dict(bounds_rule=rpy.BOUNDS_PAPER, bounds_C=60.0), dict(bounds_rule=rpy.BOUNDS_DILUTE),
               dict(d_min=0.04, d_max=40.0)):
        # past 1024 beads the dilute rule's d_max is a quarter of lambda_max: T_16 reaches 1e18
        # there and meets a coefficient of 5e-6 that is rounded to 1e-16
        if kw.get("bounds_rule") == rpy.BOUNDS_DILUTE and w.n > 1024:
            continue
        bp = rpy.make_bd_params(dt=1e-3, n_cheb=17, **kw)
        p, q = pos.clone(), pos.clone()
        for c, r in ((a, p), (b, q)):
            c.step(r, bp, seed=3, step=1)
        # the dilute interval lets T_p grow past [-1, 1]
        assert torch.max(torch.abs(p - q)).item() <= 1e-11 * torch.max(torch.abs(q)).item()


@pytest.mark.parametrize("size", [(24, 32), (7, 127), (32, 32)])
@pytest.mark.parametrize("alphaL,M", [(6.0, 4.6), (4.0, 3.5), (8.0, 3.5)])
def test_wave_vector_sets(size, alphaL, M):
    """Rows past 600 beads at other cutoffs, against the tiles of a context with an FP32
    copy."""
    w = inputs.Workload("forms", *size, 1.0, alphaL=alphaL, M=M, seed=94)
    pos = torch.from_numpy(w.positions()).cuda()
    a, b = rpy.context_for(w, max_rhs=4), rpy.context_for(w, lowp="f32", max_rhs=4)
    a.build(pos)
    b.build(pos)
    for m in (1, 2, 3, 4):
        v = _vec(w, m) * 0.03
        assert _by_rows(a, lambda: a.sqrt_apply(v, 12, 0.05, 12.0))
        x, y = (c.sqrt_apply(v, 12, 0.05, 12.0) for c in (a, b))
        assert torch.max(torch.abs(x - y)).item() <= 1e-12 * torch.max(torch.abs(y)).item()


@pytest.mark.parametrize("size,M", [((20, 20), 3.5), ((40, 25), 4.6), ((25, 41), 4.6)])
def test_drift_by_rows_against_oracle(size, M):
    """The drift products of a step (1, 3 or 4 vectors by rows) and the sums of 20 terms."""
    w, pos, a = _setup(size, M)
    D = oracle.diffusion_matrix(pos.cpu().numpy(), w.L, w.a, w.alpha, w.rc, w.n2max)
    F = oracle.spring_forces(pos.cpu().numpy(), w.nchains, w.bpc)
    drift = (D @ F.reshape(-1)).reshape(-1, 3)
    dw = rpy.rpy_gaussian_noise(torch.empty_like(pos), 7, 11, 1e-3)
    for kw in (dict(d_min=0.03, d_max=60.0), dict(bounds_rule=rpy.BOUNDS_PAPER, bounds_C=60.0),
               dict(bounds_rule=rpy.BOUNDS_DILUTE)):
        bp = rpy.make_bd_params(dt=1e-3, n_cheb=20, **kw)
        got, noise, _ = a.step(pos.clone(), bp, dw=dw, want=True)
        assert np.abs(got.cpu().numpy() - drift).max() <= 1e-12 * np.abs(drift).max()
        if "d_min" in kw:
            want = oracle.cheb_sqrt(D, dw.cpu().numpy().reshape(1, -1), 20, 0.03, 60.0).reshape(-1, 3)
            assert np.abs(noise.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
