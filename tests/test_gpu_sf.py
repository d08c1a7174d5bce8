"""The structure factors by columns of wave vectors, beside the FP32, BF16 and
FP64 tiles and in a launch of their own (low-memory form): products against
the oracle at bead counts around the workgroups' strides and at wave-vector
sets whose columns end in every remainder of the four n_z per workgroup, one
to four vectors."""
import numpy as np
import pytest
import torch

import oracle
from paper_1203_6208_amd import inputs, rpy

pytestmark = pytest.mark.gpu
# every product, with the entries it stores: 1e-12
TOL = 1e-12


def _entries(dense, prec):
    """The stored real-space entries as the product of `prec` reads them."""
    if prec == "f64":
        return dense
    d = dense.to(torch.float32)
    return (d if prec == "f32" else d.to(torch.bfloat16)).to(torch.float64)


def _run(chains, bpc, alphaL, M, m, lowp, lma):
    w = inputs.Workload("sf", chains, bpc, 1.0, alphaL=alphaL, M=M, seed=91)
    pos = torch.from_numpy(w.positions()).cuda()
    ctx = rpy.context_for(w, lowp=lowp, max_rhs=m, lma=lma)
    ctx.build(pos)
    v = np.random.default_rng(3).standard_normal((m, w.n, 3))
    vc = torch.from_numpy(v).cuda()
    p = pos.cpu().numpy()
    recip = oracle.recip_space_matrix(p, w.L, w.a, w.alpha, w.n2max)
    if lma:
        dense = torch.from_numpy(oracle.real_space_matrix(p, w.L, w.a, w.alpha, w.rc))
    else:
        dense = ctx.real_space_dense().cpu().reshape(3 * w.n, 3 * w.n)
    for prec in {"f64", lowp}:
        want = ((_entries(dense, prec).numpy() + recip) @ v.reshape(m, -1).T).T
        got = ctx.apply(vc, prec=prec).cpu().numpy().reshape(m, -1)
        assert np.abs(got - want).max() <= TOL * np.abs(want).max(), prec
    ctx.close()


@pytest.mark.parametrize("size", [(1, 5), (1, 127), (8, 16), (3, 43), (1, 257), (27, 19)])
@pytest.mark.parametrize("lowp", ["f32", "bf16"])
def test_beside_tiles(size, lowp):
    for m in (1, 4):
        _run(*size, 6.0, 3.5, m, lowp, 0)


@pytest.mark.parametrize("form", [(4.0, 3.5), (5.0, 3.5), (6.0, 4.6), (8.0, 3.5)])
def test_wave_vector_sets(form):
    for m in (1, 2, 3):
        _run(5, 27, *form, m, "f32", 0)


@pytest.mark.parametrize("size", [(8, 25), (1, 255), (2, 128), (3, 171)])
@pytest.mark.parametrize("alphaL", [12.0, 14.0])
def test_alone(size, alphaL):
    for m in (1, 3):
        _run(*size, alphaL, 3.5, m, "f64", 1)


@pytest.mark.parametrize("size", [(8, 25), (3, 64), (2, 65), (1, 255)])
@pytest.mark.parametrize("lma", [0, 1])
def test_back_projection_by_columns(size, lma):
    """More wave vectors than the staged limit: every epilogue, the fused
    trials and, with stored tiles (an FP32 copy keeps the FP64 products on
    them), the reverse mode between products."""
    w = inputs.Workload("cols", *size, 1.0, alphaL=12.0, M=3.5, seed=93)
    p = w.positions()
    pos = torch.from_numpy(p).cuda()
    kw = dict(lma=1) if lma else dict(lowp="f32", grad=1)
    ctx = rpy.context_for(w, max_rhs=3, cheb_keep=64, **kw)
    ctx.build(pos)
    D = oracle.diffusion_matrix(p, w.L, w.a, w.alpha, w.rc, w.n2max)
    lam = np.linalg.eigvalsh(D)
    lo, hi = 0.8 * lam[0], 1.2 * lam[-1]
    for m in (1, 3):
        dw = w.noise(m=m)
        ds = ctx.sqrt_apply(torch.from_numpy(dw).cuda(), 14, lo, hi)
        want = oracle.cheb_sqrt(D, dw.reshape(m, -1), 14, lo, hi)
        assert np.abs(ds.cpu().numpy().reshape(m, -1) - want).max() <= TOL * np.abs(want).max()
        if not lma:
            rng = np.random.default_rng(4)
            F, g = rng.standard_normal((w.n, 3)), rng.standard_normal((w.n, 3))
            f1 = dw[:1].reshape(w.n, 3)
            gp, gF = torch.empty_like(pos), torch.empty_like(pos)
            c = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (F, f1, g)]
            rpy.rpy_u_vjp(ctx.handle, pos, *c, 8, lo, hi, gp, gF, None)
            wp, wF = oracle.u_vjp(p, w.L, w.a, w.alpha, w.rc, w.n2max, F, f1, g, 8, lo, hi)
            # dL/dR: a sum of terms of both signs, as every test of the reverse mode
            assert np.abs(gp.cpu().numpy() - wp).max() <= 1e-10 * np.abs(wp).max()
            assert np.abs(gF.cpu().numpy() - wF).max() <= TOL * np.abs(wF).max()
        ds, ef, n = ctx.sqrt_adaptive(torch.from_numpy(dw).cuda(), lo, hi, 1e-3, 64)
        n_o, want = oracle.cheb_adaptive(D, dw.reshape(m, -1), lo, hi, 1e-3, 64)
        assert n == n_o
        assert np.abs(ds.cpu().numpy().reshape(m, -1) - want).max() <= TOL * np.abs(want).max()
    ctx.close()


@pytest.mark.parametrize("size", [(32, 64), (3, 683), (41, 51)])
def test_back_projection_groups(size):
    """Eight beads per workgroup up to 2048 beads, 16 above: products and adaptive
    series (whose trials' partial sums are per workgroup) of one and three
    vectors against the block path of five, which has workgroups of its own."""
    w = inputs.Workload("groups", *size, 1.0, seed=94)
    pos = torch.from_numpy(w.positions()).cuda()
    a = rpy.context_for(w, lowp="bf16", max_rhs=5, cheb_keep=64)
    a.build(pos)
    v = torch.from_numpy(np.random.default_rng(6).standard_normal((5, w.n, 3))).cuda()
    want, (ws, wf, wn) = a.apply(v), a.sqrt_adaptive(v, 0.04, 40.0, 1e-2, 64)
    for m in (1, 3):
        got = a.apply(v[:m])
        assert (got - want[:m]).abs().max().item() <= TOL * want.abs().max().item()
        gs, gf, gn = a.sqrt_adaptive(v[:m], 0.04, 40.0, 1e-2, 64, n_start=wn)
        assert gn == wn
        assert (gs - ws[:m]).abs().max().item() <= TOL * ws.abs().max().item()
