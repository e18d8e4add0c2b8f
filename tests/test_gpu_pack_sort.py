"""cube2_pack's sort against a stable argsort of the cell keys, bit for bit.

The cases take both ways of sorting (by tile and then by cell; by the whole key
where there are few particles per tile or one tile), one and two digits, of 8
and 9 bits, a last block of one key, a full one and one more than full, every
particle in one cell or one tile (long runs of empty tiles), and ties in input
order (several particles at one position)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(x, n_fine):
    import paper_2512_12629_amd as m
    x = np.ascontiguousarray(x).astype(np.float32)
    x[x >= 1.0] = 0.0
    n = x.shape[1]
    c = m.Cube2(m.Config(n_fine=n_fine), n_max=n)
    q = np.floor(x.astype(np.float64) * n_fine * 32768.0).astype(np.int64)
    cell = q >> 16
    t, u, nt = cell >> 3, cell & 7, n_fine // 16
    key = ((t[2] * nt + t[1]) * nt + t[0]) * 512 + (u[2] * 8 + u[1]) * 8 + u[0]
    order = np.argsort(key, kind="stable")
    for _ in range(2):
        pos, cs, perm = c.pack(torch.from_numpy(x).cuda())
        assert np.array_equal(perm.cpu().numpy(), order)
        assert np.array_equal(pos.cpu().numpy().view(np.uint16), (q & 0xFFFF)[:, order])
        assert np.array_equal(cs.cpu().numpy().view(np.uint32),
                              np.searchsorted(key[order], np.arange((n_fine // 2) ** 3 + 1)))


@pytest.mark.parametrize("n_fine,n", [(16, 1), (16, 900), (32, 511), (32, 512), (32, 4097), (64, 4096),
                                      (64, 60001), (128, 32769), (256, 300000), (512, 2100000),
                                      (512, 5000), (1024, 40000)])
def test_uniform_positions(n_fine, n):
    rng = np.random.default_rng(n)
    x = rng.random((3, n))
    x[:, n // 2:] = x[:, :n - n // 2][:, ::-1]      # ties far apart in the input
    _check(x, n_fine)


@pytest.mark.parametrize("n_fine,n", [(64, 20000), (512, 2100000)])
def test_everything_in_one_tile(n_fine, n):
    rng = np.random.default_rng(n)
    _check((16.0 * 2 + 16.0 * rng.random((3, n))) / n_fine, n_fine)
    _check(0.5 + np.zeros((3, n)), n_fine)


def test_largest_mesh_by_tile():
    """64^3 tiles: two digits of 9 bits."""
    n = 64 * 64 ** 3 + 5
    x = torch.rand((3, n), generator=torch.Generator().manual_seed(1)).numpy()
    _check(x, 1024)
