"""cube2_kick_drift's re-sort against a stable argsort, bit for bit: positions,
cell starts, velocities and permutation, for the drift in FP64 with separately
rounded operations.

The cases take both ways of sorting: the local one (particles stay within the
neighbouring tiles), at one, two and four tiles per axis, with a tile of one
chunk (1024 particles), one more and many, and empty tiles; the radix sort
where a single particle goes farther, where all do, and where there are too few
particles per tile for the local one; and steps that do not move at all."""
import numpy as np
import pytest

from helpers import ios_decode

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _key(q, n_fine):
    c = q >> 16
    t, u = c >> 3, c & 7
    nt = n_fine // 16
    return ((t[2] * nt + t[1]) * nt + t[0]) * 512 + (u[2] * 8 + u[1]) * 8 + u[0]


def _check(x, n_fine, move, far=0, bad=0, seed=1):
    import paper_2512_12629_amd as m
    rng = np.random.default_rng(seed)
    x = np.ascontiguousarray(x).astype(np.float32)
    n = x.shape[1]
    c = m.Cube2(m.Config(n_fine=n_fine), n_max=n)
    pos, cs, _ = c.pack(torch.from_numpy(x).cuda())
    q = ios_decode(pos.cpu().numpy().view(np.uint16), cs.cpu().numpy().view(np.uint32), n_fine)
    vel = (move * rng.standard_normal((3, n))).astype(np.float32)
    acc = (move * rng.standard_normal((3, n))).astype(np.float32)
    for k in range(far):
        vel[k % 3, rng.integers(n)] = 0.6 * n_fine
    for k in range(bad):
        acc[k % 3, rng.integers(n)] = (np.nan, np.inf)[k % 2]
    kick, drift = 0.37, 1.0
    with np.errstate(all="ignore"):
        v1 = vel.astype(np.float64) + kick * acc.astype(np.float64)
        dq = np.rint(drift * v1 * 32768.0)
        ok = np.abs(dq) < 2.0 ** 62
    q1 = (q + np.where(ok, dq, 0.0).astype(np.int64)) % (n_fine * 32768)
    key = _key(q1, n_fine)
    order = np.argsort(key, kind="stable")
    for _ in range(2):
        p2, cs2, v2, perm = c.kick_drift(pos, cs, torch.from_numpy(vel).cuda(),
                                         torch.from_numpy(acc).cuda(), kick, drift)
        assert np.array_equal(perm.cpu().numpy(), order)
        assert np.array_equal(cs2.cpu().numpy().view(np.uint32),
                              np.searchsorted(key[order], np.arange((n_fine // 2) ** 3 + 1)))
        assert np.array_equal(p2.cpu().numpy().view(np.uint16), (q1 & 0xFFFF)[:, order])
        with np.errstate(all="ignore"):
            want = v1.astype(np.float32)[:, order]
        got = v2.cpu().numpy()
        assert np.array_equal(got.view(np.uint32)[~np.isnan(want)], want.view(np.uint32)[~np.isnan(want)])
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert c.status() == (-7 if bad else 0)


@pytest.mark.parametrize("n_fine,n", [(16, 40), (16, 5000), (32, 300), (32, 9000), (64, 2100), (64, 70000),
                                      (64, 50)])
@pytest.mark.parametrize("move", [0.0, 0.3, 4.0])
def test_uniform(n_fine, n, move):
    _check(np.random.default_rng(n).random((3, n)), n_fine, move)


@pytest.mark.parametrize("far", [1, 500])
def test_particles_beyond_the_neighbouring_tiles(far):
    _check(np.random.default_rng(far).random((3, 30000)), 128, 0.3, far=far)


@pytest.mark.parametrize("count", [1023, 1024, 1025, 2048, 7000])
def test_dense_tile_beside_empty_ones(count):
    rng = np.random.default_rng(count)
    x = np.concatenate([0.25 + 0.25 * rng.random((3, count)), rng.random((3, 1000)) * 0.2], axis=1)
    _check(x, 64, 1.0)


def test_one_cell_holds_everything_and_bad_accelerations():
    rng = np.random.default_rng(3)
    _check(0.5 + rng.random((3, 3000)) / 64.0, 64, 0.0)
    _check(rng.random((3, 20000)), 64, 0.5, bad=4)
