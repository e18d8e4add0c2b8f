"""cube2_pack and cube2_kick_drift where tiles hold more particles than one workgroup sorts
(8192): one such tile or several, spread, in one cell, at the limit and at multiples of
it, in the first and the last tile; bit for bit against a stable argsort.  And they must
not cost the sort of everything else many times over."""
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


def _clump(rng, n_fine, count, at, size, rest):
    x = np.concatenate([at[:, None] + size * rng.random((3, count)), n_fine * rng.random((3, rest))], axis=1)
    return rng.permutation(x.T).T / n_fine


def _check(x, n_fine, far=0):
    import paper_2512_12629_amd as m
    rng = np.random.default_rng(1)
    x = np.ascontiguousarray(x).astype(np.float32)
    n = x.shape[1]
    c = m.Cube2(m.Config(n_fine=n_fine), n_max=n)
    pos, cs, perm = c.pack(torch.from_numpy(x).cuda())
    q0 = np.floor(x.astype(np.float64) * (n_fine * 32768)).astype(np.int64) % (n_fine * 32768)
    key = _key(q0, n_fine)
    order = np.argsort(key, kind="stable")
    cells = np.arange((n_fine // 2) ** 3 + 1)
    assert np.array_equal(perm.cpu().numpy(), order)
    assert np.array_equal(cs.cpu().numpy().view(np.uint32), np.searchsorted(key[order], cells))
    assert np.array_equal(pos.cpu().numpy().view(np.uint16), (q0 & 0xFFFF)[:, order])
    q = ios_decode(pos.cpu().numpy().view(np.uint16), cs.cpu().numpy().view(np.uint32), n_fine)
    vel = (0.4 * rng.standard_normal((3, n))).astype(np.float32)
    acc = (0.4 * rng.standard_normal((3, n))).astype(np.float32)
    for k in range(far):
        vel[k % 3, rng.integers(n)] = 0.5 * n_fine
    v1 = vel.astype(np.float64) + 0.37 * acc.astype(np.float64)
    q1 = (q + np.rint(v1 * 32768.0).astype(np.int64)) % (n_fine * 32768)
    key = _key(q1, n_fine)
    order = np.argsort(key, kind="stable")
    for _ in range(2):
        p2, cs2, v2, perm = c.kick_drift(pos, cs, torch.from_numpy(vel).cuda(), torch.from_numpy(acc).cuda(),
                                         0.37, 1.0)
        assert np.array_equal(perm.cpu().numpy(), order)
        assert np.array_equal(cs2.cpu().numpy().view(np.uint32), np.searchsorted(key[order], cells))
        assert np.array_equal(p2.cpu().numpy().view(np.uint16), (q1 & 0xFFFF)[:, order])
        assert np.array_equal(v2.cpu().numpy(), v1.astype(np.float32)[:, order])
        assert c.status() == 0


@pytest.mark.parametrize("count", [8191, 8192, 8193, 16384, 16385, 70000])
@pytest.mark.parametrize("size", [15.9, 1.9])
def test_one_heavy_tile(count, size):
    _check(_clump(np.random.default_rng(count), 64, count, np.array([32.0, 16.0, 48.0]), size, 6000), 64)


def test_first_and_last_tile_and_far_particles():
    rng = np.random.default_rng(3)
    a = _clump(rng, 128, 20000, np.array([0.0, 0.0, 0.0]), 15.9, 30000)
    b = _clump(rng, 128, 9000, np.array([112.0, 112.0, 112.0]), 15.9, 0)
    d = _clump(rng, 128, 300000, np.array([64.0, 80.0, 16.0]), 7.9, 0)
    _check(np.concatenate([a, b, d], axis=1), 128, far=3)


def test_all_tiles_heavy():
    _check(np.random.default_rng(4).random((3, 90000)), 32)
    _check(np.random.default_rng(5).random((3, 30000)), 16)


def test_a_heavy_tile_costs_little():
    import paper_2512_12629_amd as m

    def time(heavy):
        rng = np.random.default_rng(6)
        x = _clump(rng, 256, heavy, np.array([128.0, 64.0, 32.0]), 14.0, (1 << 21) - heavy).astype(np.float32)
        x = torch.from_numpy(np.ascontiguousarray(x)).cuda() % 1.0
        c = m.Cube2(m.Config(n_fine=256), n_max=x.shape[1])
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                c.pack(x)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    assert time(1 << 17) <= 3.0 * time(0)
