"""The PP kernels' two kinds of tiles, side by side: light ones, which waves
take in pairs of cell layers (single layers on small meshes), and the others,
which whole workgroups take, against the oracle for the force and its adjoint.

The cases put their densities at the edges: every tile light, none, both in one
mesh; on the smallest mesh (one tile, all its neighbours itself), on one whose
items outnumber the waves (claimed in chunks) and with a two-layer box at the
staging capacity of the forward (520 particles) and of the adjoint (512), one
below it and one above.  Bar as in the other PP tests: median 1e-4, p99 1e-3
relative to max(|F|, 1e-6 median |F|)."""
import numpy as np
import pytest

import oracle
from helpers import ios_decode

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _stats(got, ref):
    fr = np.linalg.norm(ref, axis=0)
    has = fr > 0
    if not has.any():
        return 0.0, 0.0
    e = np.linalg.norm(got - ref, axis=0)[has] / np.maximum(fr[has], 1e-6 * np.median(fr[has]))
    return float(np.median(e)), float(np.percentile(e, 99))


def _run(x, n_fine, seed):
    import paper_2512_12629_amd as m
    x = np.ascontiguousarray(x).astype(np.float32)
    c = m.Cube2(m.Config(n_fine=n_fine), n_max=x.shape[1])
    pos, cs, _ = c.pack(torch.from_numpy(x).cuda())
    q = ios_decode(pos.cpu().numpy().view(np.uint16), cs.cpu().numpy().view(np.uint32), n_fine)
    o = oracle.Oracle(oracle.Params(n_fine=n_fine, coarse_ratio=0))
    ab = np.random.default_rng(seed).standard_normal(x.shape).astype(np.float32)
    xf = q / 2.0 ** 15
    for got, ref in ((c.pp_force(pos, cs), o.pp_accel(xf)),
                     (c.pp_force_backward(pos, cs, torch.from_numpy(ab).cuda()),
                      o.pp_adjoint(xf, ab.astype(np.float64)))):
        med, p99 = _stats(got.double().cpu().numpy(), ref)
        assert med < 1e-4 and p99 < 1e-3, (med, p99)


@pytest.mark.parametrize("n_fine,n,dense", [(16, 1, 0), (16, 300, 0), (16, 3000, 0), (32, 4096, 0),
                                            (64, 20000, 3000), (64, 5, 0), (256, 400000, 2000)])
def test_light_and_heavy_tiles(n_fine, n, dense):
    rng = np.random.default_rng(n_fine + n)
    x = rng.random((3, n))
    if dense:      # a clump across the corner of eight tiles
        x[:, :dense] = 0.5 + (rng.random((3, dense)) - 0.5) * 6.0 / n_fine
    _run(x, n_fine, n)


@pytest.mark.parametrize("count", [511, 512, 513, 519, 520, 521])
def test_boxes_at_the_staging_capacity(count):
    """`count` particles in the cells of tile (1, 1, 1)'s lowest two layers
    (and none in its halo), so that its lowest two-layer box holds exactly so
    many."""
    rng = np.random.default_rng(count)
    lo, size = np.array([[16.0], [16.0], [16.0]]), np.array([[16.0], [16.0], [4.0]])
    _run((lo + size * rng.random((3, count))) / 64.0, 64, count)
