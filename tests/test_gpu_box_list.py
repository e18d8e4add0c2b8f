"""The particles of a box of cells as one list, found by counting bits in spans of
4096 positions (mass assignment and the fine cotangent scatter): cells that
begin, end or lie across a span, empty cells and empty boxes.  Densities are
integers, equal to the oracle's; the PM adjoint against the oracle, median 1e-4
and p99 1e-3 relative to max(|F|, 1e-6 median |F|).

The sum of PM and PP formed by the last PM kernel: the same additions in the same
order as PM, then PP, by themselves, so equal bit for bit.

The gather of a tile's box, whose cells of more than 64 particles are copied by a
whole wave: equal to a copy on the host."""
import numpy as np
import pytest

import oracle
from helpers import ios_decode

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _stats(got, ref):
    fr = np.linalg.norm(ref, axis=0)
    has = fr > 0
    e = np.linalg.norm(got - ref, axis=0)[has] / np.maximum(fr[has], 1e-6 * np.median(fr[has]))
    return float(np.median(e)), float(np.percentile(e, 99))


def _cells(rng, counts, around):
    """counts[i] particles in the i-th IOS cell (2 fine cells) from (20, 20, 20) on
    along x, and `around` anywhere in the 128^3 box."""
    x = [np.array([[20.0 + 2 * i], [20.0], [20.0]]) + 1.99 * rng.random((3, k)) for i, k in enumerate(counts)]
    x = np.concatenate(x + [127.9 * rng.random((3, around))], axis=1) / 128.0
    return np.ascontiguousarray(x).astype(np.float32)


@pytest.mark.parametrize("assign", ["cic", "tsc"])
@pytest.mark.parametrize("counts,around", [((1,), 0), ((4096,), 0), ((4095, 1, 3), 0), ((4097, 5), 0),
                                           ((64, 4032, 64), 0), ((9000, 0, 4096), 700)])
def test_spans(counts, around, assign):
    import paper_2512_12629_amd as m
    rng = np.random.default_rng(sum(counts))
    x = _cells(rng, counts, around)
    tsc = assign == "tsc"
    c = m.Cube2(m.Config(n_fine=128, coarse_ratio=4, flags=m.CUBE2_ASSIGN_TSC if tsc else 0),
                n_max=x.shape[1])
    pos, cs, _ = c.pack(torch.from_numpy(x).cuda())
    xf = ios_decode(pos.cpu().numpy().view(np.uint16), cs.cpu().numpy().view(np.uint32), 128) / 2.0 ** 15
    p = 3 if tsc else 2
    for level, (n, H) in enumerate(((128, 1), (32, 4))):
        _, fx = c.deposit(pos, cs, level, fx=True)
        assert np.array_equal(fx.cpu().numpy().astype(np.int64),
                              oracle.deposit_fx(xf, n, H, p).astype(np.int64)), level
    if x.shape[1] == 1:
        return    # a particle's force on itself is zero wherever it is: so is its adjoint
    o = oracle.Oracle(oracle.Params(n_fine=128, coarse_ratio=4, assign=p))
    ab = rng.standard_normal(x.shape).astype(np.float32)
    got = c.pm_force_backward(pos, cs, torch.from_numpy(ab).cuda()).double().cpu().numpy()
    med, p99 = _stats(got, o.pm_adjoint(xf, ab.astype(np.float64)))
    assert med < 1e-4 and p99 < 1e-3, (med, p99)


@pytest.mark.parametrize("n_fine,ratio", [(64, 0), (128, 0), (128, 4)])
@pytest.mark.parametrize("n", [1, 255, 30001])
def test_sum_of_pm_and_pp(n_fine, ratio, n):
    import paper_2512_12629_amd as m
    rng = np.random.default_rng(n)
    x = torch.from_numpy(np.ascontiguousarray(rng.random((3, n)).astype(np.float32) * 0.999)).cuda()
    c = m.Cube2(m.Config(n_fine=n_fine, coarse_ratio=ratio), n_max=n)
    pos, cs, _ = c.pack(x)
    assert torch.equal(c.force(pos, cs), c.pm_force(pos, cs) + c.pp_force(pos, cs))
    ab = torch.from_numpy(rng.standard_normal((3, n)).astype(np.float32)).cuda()
    x0 = torch.from_numpy(rng.standard_normal((3, n)).astype(np.float32)).cuda()
    pm, pp = c.pm_force_backward(pos, cs, ab), c.pp_force_backward(pos, cs, ab)
    assert torch.equal(c.force_backward(pos, cs, ab), pm + pp)
    assert torch.equal(c.force_backward(pos, cs, ab, x0.clone()), (x0 + pm) + pp)


@pytest.mark.parametrize("counts", [(63, 64, 65), (1, 127, 128, 129, 0, 2000)])
def test_gather_of_dense_cells(counts):
    import paper_2512_12629_amd as m
    rng = np.random.default_rng(len(counts))
    x = _cells(rng, counts, 20000)
    t = m.Cube2Tiled(m.Config(n_fine=128, coarse_ratio=4), 16, 8, x.shape[1])
    pos, cs, _ = t.g.pack(torch.from_numpy(x).cuda())
    t._local(x.shape[1])
    mc = m.cube2_tile_gather(t.g.ctx, pos, cs, [(16, 16, 16)], 16, 8, t.x_buf, t.i_buf, t.g.work)
    got = t.x_buf[:3 * mc].view(3, mc).cpu().numpy()
    idx = t.i_buf[:mc].cpu().numpy().astype(np.int64)
    q = ios_decode(pos.cpu().numpy().view(np.uint16), cs.cpu().numpy().view(np.uint32), 128)
    rel = q - (8 << 15)                      # the box: fine cells 8 .. 40 per axis
    inside = np.all((rel >= 0) & (rel < (32 << 15)), axis=0)
    cell = np.floor_divide(rel, 1 << 16)
    order = np.lexsort((np.arange(x.shape[1]), cell[0], cell[1], cell[2]))
    want = order[inside[order]]
    assert np.array_equal(idx, want)
    assert np.array_equal(got, (rel[:, want] / float(32 << 15)).astype(np.float32))


@pytest.mark.parametrize("b_fine,b_pp", [(2.0, 0.2), (3.5, 0.0625)])
@pytest.mark.parametrize("counts,around", [((1,), 0), ((2, 0, 511), 0), ((4096,), 1), ((4097, 600), 3000)])
def test_pp_force_f64_spans(counts, around, b_fine, b_pp):
    """The FP64 PP force, whose box is staged in the same spans, against the oracle's
    (both FP64: the bars of the FP64 form's own tests)."""
    import paper_2512_12629_amd as m
    rng = np.random.default_rng(sum(counts))
    x = _cells(rng, counts, around)
    c = m.Cube2(m.Config(n_fine=128, b_fine=b_fine, b_pp=b_pp, flags=m.CUBE2_FP64_FORM),
                n_max=x.shape[1])
    pos, cs, _ = c.pack(torch.from_numpy(x).cuda())
    xf = ios_decode(pos.cpu().numpy().view(np.uint16), cs.cpu().numpy().view(np.uint32), 128) / 2.0 ** 15
    got = c.pp_force_f64(pos, cs).cpu().numpy()
    ref = oracle.Oracle(oracle.Params(n_fine=128, b_fine=b_fine, b_pp=b_pp)).pp_accel(xf)
    has = np.linalg.norm(ref, axis=0) > 0
    assert np.all(got[:, ~has] == 0)
    if has.any():
        med, p99 = _stats(got, ref)
        assert med < 1e-12 and p99 < 1e-10, (med, p99)
