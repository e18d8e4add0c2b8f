"""The PP kernels where all heavy tiles are split into whole blocks (forward; from 1025
to 2048 of them) or none but the heaviest are, and waves whose lanes meet a dense cell
in different neighbour rows.  Force and adjoint against the oracle, median 1e-4 and p99
1e-3 relative to max(|F|, 1e-6 median |F|)."""
import numpy as np
import pytest

import oracle
from helpers import ios_decode

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(x, n_fine, b_fine=2.0, b_pp=0.2):
    import paper_2512_12629_amd as m
    rng = np.random.default_rng(3)
    x = np.ascontiguousarray(x).astype(np.float32)
    c = m.Cube2(m.Config(n_fine=n_fine, b_fine=b_fine, b_pp=b_pp), n_max=x.shape[1])
    pos, cs, _ = c.pack(torch.from_numpy(x).cuda())
    xf = ios_decode(pos.cpu().numpy().view(np.uint16), cs.cpu().numpy().view(np.uint32), n_fine) / 2.0 ** 15
    o = oracle.Oracle(oracle.Params(n_fine=n_fine, coarse_ratio=0, b_fine=b_fine, b_pp=b_pp))
    ab = rng.standard_normal(x.shape).astype(np.float32)
    for got, ref in ((c.pp_force(pos, cs), o.pp_accel(xf)),
                     (c.pp_force_backward(pos, cs, torch.from_numpy(ab).cuda()),
                      o.pp_adjoint(xf, ab.astype(np.float64)))):
        got = got.double().cpu().numpy()
        fr = np.linalg.norm(ref, axis=0)
        has = fr > 0
        e = np.linalg.norm(got - ref, axis=0)[has] / np.maximum(fr[has], 1e-6 * np.median(fr[has]))
        assert np.median(e) < 1e-4 and np.percentile(e, 99) < 1e-3, (np.median(e), np.percentile(e, 99))


@pytest.mark.parametrize("tiles", [1025, 2048, 2049])
def test_many_heavy_tiles(tiles):
    """One dense cell in the middle of each of `tiles` tiles of 16^3 of them: the box
    of the two z-layers around it is beyond the light tiles' in each."""
    rng = np.random.default_rng(tiles)
    t = rng.permutation(4096)[:tiles]
    at = 16.0 * np.stack([t % 16, t // 16 % 16, t // 256]) + 8.0
    x = np.repeat(at, 540, axis=1) + 1.9 * rng.random((3, 540 * tiles))
    _check(np.concatenate([x, 255.9 * rng.random((3, 20000))], axis=1) / 256.0, 256)


@pytest.mark.parametrize("b_fine,b_pp", [(2.0, 0.2), (3.5, 0.0625)])
@pytest.mark.parametrize("dense", [1, 600, 5000])
def test_dense_cell_among_sparse(dense, b_fine, b_pp):
    """One particle per cell around one cell of `dense`."""
    rng = np.random.default_rng(dense)
    g = np.stack(np.meshgrid(*[np.arange(32)] * 3, indexing="ij")).reshape(3, -1)
    x = 2.0 * g + 1.9 * rng.random(g.shape)
    y = np.array([[30.0], [16.0], [40.0]]) + 1.9 * rng.random((3, dense))
    _check(np.concatenate([x, y], axis=1) / 64.0, 64, b_fine, b_pp)
