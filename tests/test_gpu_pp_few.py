"""The PP kernels where heavy tiles are few: four lanes per particle, each taking
every fourth neighbour, and parts of a quarter of a block.  Counts of own
particles and neighbours around a quarter block (128 and 256 particles, forward
and adjoint), with boxes staged at once and in parts, and the tiled force whose
pair sums outside the tile proper are left out.  Force and adjoint against the
oracle, median 1e-4 and p99 1e-3 relative to max(|F|, 1e-6 median |F|)."""
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


@pytest.mark.parametrize("b_fine,b_pp", [(2.0, 0.2), (3.5, 0.0625)])
@pytest.mark.parametrize("own,cell", [(1, 700), (127, 700), (129, 700), (257, 700), (1100, 3), (4700, 1)])
def test_few_heavy_tiles(own, cell, b_fine, b_pp):
    """`own` particles in tile (1, 1, 1) of a 64^3 mesh (all of it, or one IOS
    cell for the large counts' clumps) and `cell` in one cell of its halo."""
    import paper_2512_12629_amd as m
    rng = np.random.default_rng(own)
    x = np.concatenate([16.0 + 16.0 * rng.random((3, own)),
                        np.array([[14.0], [20.0], [20.0]]) + 2.0 * rng.random((3, cell)),
                        64.0 * rng.random((3, 500))], axis=1) / 64.0
    x = np.ascontiguousarray(x).astype(np.float32)
    c = m.Cube2(m.Config(n_fine=64, b_fine=b_fine, b_pp=b_pp), n_max=x.shape[1])
    pos, cs, _ = c.pack(torch.from_numpy(x).cuda())
    xf = ios_decode(pos.cpu().numpy().view(np.uint16), cs.cpu().numpy().view(np.uint32), 64) / 2.0 ** 15
    o = oracle.Oracle(oracle.Params(n_fine=64, coarse_ratio=0, b_fine=b_fine, b_pp=b_pp))
    ab = rng.standard_normal(x.shape).astype(np.float32)
    for got, ref in ((c.pp_force(pos, cs), o.pp_accel(xf)),
                     (c.pp_force_backward(pos, cs, torch.from_numpy(ab).cuda()),
                      o.pp_adjoint(xf, ab.astype(np.float64)))):
        med, p99 = _stats(got.double().cpu().numpy(), ref)
        assert med < 1e-4 and p99 < 1e-3, (med, p99)


@pytest.mark.parametrize("tile,buffer", [(32, 16), (16, 24), (8, 12)])
def test_tiled_force_leaves_no_own_particle_out(tile, buffer):
    """Tiles whose edges lie on and off the PP tiles' (16 cells): every particle's
    pair sum is there, so that the tiled force is the local boxes' own."""
    import paper_2512_12629_amd as m
    rng = np.random.default_rng(tile)
    x = np.ascontiguousarray(rng.random((3, 30000))).astype(np.float32)
    cfg = m.Config(n_fine=64, coarse_ratio=4, b_coarse=8.0)
    t = m.Cube2Tiled(cfg, tile, buffer, x.shape[1])
    pos, cs, _ = t.g.pack(torch.from_numpy(x).cuda())
    got = t.force(pos, cs)
    t.skip.zero_()                      # every tile of the local boxes
    assert torch.equal(t.force(pos, cs), got)
