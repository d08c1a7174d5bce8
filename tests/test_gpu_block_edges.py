"""Edges of the block product's launches (5 to 16 vectors)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

from paper_1203_6208_amd import inputs, rpy  # noqa: E402


def _cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


@pytest.mark.parametrize("size", [(1, 17), (1, 127), (3, 43), (1, 257), (32, 64), (3, 683), (41, 51)])
@pytest.mark.parametrize("m", [5, 16])
def test_block_edges(size, m):
    """FP64 block products and a short series at bead counts around the groups of
    beads, chunks and workgroups of the reciprocal sum (one component per
    workgroup up to 2048 beads, three above; 8 or 16 quads per wave), against
    the vector-unit path four vectors at a time: both agree with the oracle to
    1e-12 of the largest entry."""
    w = inputs.Workload("bedge", *size, 1.0, seed=55)
    pos = _cuda(w.positions())
    a, b = (rpy.context_for(w, lowp="bf16", max_rhs=r) for r in (16, 4))
    a.build(pos)
    b.build(pos)
    v = _cuda(np.random.default_rng(8).standard_normal((m, w.n, 3)))
    for f in (lambda c, x: c.apply(x), lambda c, x: c.sqrt_apply(x, 6, 0.05, 12.0)):
        got = f(a, v)
        want = torch.cat([f(b, v[j:j + 4]) for j in range(0, m, 4)])
        assert (got - want).abs().max().item() <= 1e-12 * want.abs().max().item()


def test_tile_array_past_the_cache():
    """FP64 tiles of more than the part of the cache they may keep (some tiles read
    with allocating loads, the rest without), against a context whose FP32 copy
    has the cache: the loads differ, the arithmetic does not."""
    w = inputs.Workload("hot", 50, 59, 1.0, seed=56)   # 2950 beads: 47 x 48 / 2 tiles of 196 KB, 222 MB
    pos = _cuda(w.positions())
    a, b = rpy.context_for(w, max_rhs=16), rpy.context_for(w, lowp="f32", max_rhs=16)
    a.build(pos)
    b.build(pos)
    for m in (1, 2, 3, 4, 7, 16):
        v = _cuda(np.random.default_rng(m).standard_normal((m, w.n, 3)))
        assert torch.equal(a.apply(v), b.apply(v)), m


@pytest.mark.parametrize("size", [(20, 50), (23, 59), (30, 61), (43, 47)])
def test_runs_of_tiles(size):
    """FP64 row products summed over a workgroup's run of tiles: tile counts below,
    around and above the workgroups (136, 253, 435 and 528 tiles on 256), runs that
    end inside, at the end of and beyond a row, against the vector-unit path."""
    w = inputs.Workload("runs", *size, 1.0, seed=57)
    pos = _cuda(w.positions())
    a, b = rpy.context_for(w, max_rhs=16), rpy.context_for(w, lowp="f32", max_rhs=4)
    a.build(pos)
    b.build(pos)
    for m in (5, 16):
        v = _cuda(np.random.default_rng(m).standard_normal((m, w.n, 3)))
        got = a.apply(v)
        want = torch.cat([b.apply(v[j:j + 4]) for j in range(0, m, 4)])
        assert (got - want).abs().max().item() <= 1e-12 * want.abs().max().item()
        assert torch.equal(got, a.apply(v))
