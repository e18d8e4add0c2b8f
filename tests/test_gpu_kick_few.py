"""cube2_kick_drift on one or two tiles per axis (the local re-sort alone), with particles on
either side of its limits (128 per tile; 8192 in one tile), and with particles that leave
the neighbouring tiles above the first: bit for bit against a stable argsort.  And with few
particles per tile a step must not cost many times their sort."""
import numpy as np
import pytest

from test_gpu_kick_far import _check, _state

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_fine", [16, 32])
@pytest.mark.parametrize("n", [1, 2, 64, 1023, 8191, 8192, 8193])
@pytest.mark.parametrize("scale", [1.0, 40.0])
def test_one_and_two_tiles_per_axis(n_fine, n, scale):
    _, c, pos, cs, q, vel = _state(n, n_fine, n)
    _check(c, pos, cs, q, scale * vel, n_fine)


def test_no_particles():
    import paper_2512_12629_amd as m
    for n_fine in (16, 32, 64):
        c = m.Cube2(m.Config(n_fine=n_fine), n_max=1)
        pos, cs, _ = c.pack(torch.empty((3, 0), device="cuda"))
        v = torch.empty((3, 0), device="cuda")
        _, cs2, _, _ = c.kick_drift(pos, cs, v, v, 0.5, 1.0)
        assert not cs2.any()


@pytest.mark.parametrize("n_fine", [64, 128])
@pytest.mark.parametrize("per_tile", [127, 128, 130])
@pytest.mark.parametrize("far", [0, 1, 2048, 2049])
def test_far_particles_about_the_limit(n_fine, per_tile, far):
    n = per_tile * (n_fine // 16) ** 3
    rng, c, pos, cs, q, vel = _state(n, n_fine, far)
    vel[0, rng.permutation(n)[:far]] = 0.5 * n_fine
    _check(c, pos, cs, q, vel, n_fine)


@pytest.mark.parametrize("into", [5, 32, 33])
def test_into_one_tile(into):
    n_fine = 64
    rng, c, pos, cs, q, vel = _state(130 * 64, n_fine, into)
    pick = rng.permutation(np.nonzero(np.all(q >> 19 == 0, axis=0))[0])[:into]
    to = 35.0 + 9.0 * rng.random((into, 3))
    vel[:, pick] = (to.T - q[:, pick] / 32768.0).astype(np.float32)
    _check(c, pos, cs, q, vel, n_fine)


def test_few_particles_cost_little():
    import paper_2512_12629_amd as m

    def time(f):
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                f()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    n = 104 ** 3
    x = torch.from_numpy(np.random.default_rng(1).random((3, n)).astype(np.float32)).cuda()
    c = m.Cube2(m.Config(n_fine=512), n_max=n)
    pos, cs, _ = c.pack(x)
    v = 0.3 * torch.randn((3, n), device="cuda")
    assert time(lambda: c.kick_drift(pos, cs, v, v, 0.1, 1.0)) <= 1.6 * time(lambda: c.pack(x))
