"""cube2_pack and cube2_kick_drift where a tile holds about as many particles as the sorts
and the drift give to one workgroup (4096; 8192 in the drift of more than a million) and
as the chunks change at (2048 to 65536 particles of a tile, then 8192), bit for bit against
a stable argsort.  And one such tile must not cost as much as everything else."""
import numpy as np
import pytest

from test_gpu_heavy_tiles_sort import _check, _clump

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [4095, 4096, 4097, 6144, 6145, 65536, 65537, 73729])
@pytest.mark.parametrize("size", [15.9, 1.9])
def test_one_tile_about_the_limits(count, size):
    rng = np.random.default_rng(count)
    # (the others elsewhere, so that the tile has exactly `count` before the step)
    x = _clump(rng, 64, count, np.array([32.0, 16.0, 48.0]), size, 0)
    rest = rng.random((3, 9000)) * np.array([[1.0], [1.0], [0.5]])
    _check(np.concatenate([rest, x], axis=1), 64)
    _check(x, 64)


@pytest.mark.parametrize("n_fine,n", [(16, 4096), (16, 4097), (32, 4096), (32, 4097), (32, 40000)])
def test_few_tiles(n_fine, n):
    _check(np.random.default_rng(n).random((3, n)), n_fine)


@pytest.mark.parametrize("n", [1 << 20, (1 << 20) + 1])
def test_about_a_million(n):
    rng = np.random.default_rng(n)
    x = _clump(rng, 128, 6000, np.array([64.0, 80.0, 16.0]), 7.9, n - 6000)
    _check(x, 128, far=2)


def test_heavy_tiles_all_over_a_large_mesh():
    rng = np.random.default_rng(7)
    x = [_clump(rng, 256, 4500 + 700 * k, 16.0 * rng.integers(0, 16, 3), 15.9, 0) for k in range(12)]
    _check(np.concatenate(x + [rng.random((3, 140 * 16 ** 3))], axis=1), 256, far=1)


def test_a_heavy_tile_costs_little():
    import paper_2512_12629_amd as m

    def time(heavy):
        rng = np.random.default_rng(6)
        x = _clump(rng, 64, heavy, np.array([32.0, 16.0, 48.0]), 1.9, 130000 - heavy).astype(np.float32)
        x = torch.from_numpy(np.ascontiguousarray(x)).cuda() % 1.0
        c = m.Cube2(m.Config(n_fine=64), n_max=x.shape[1])
        pos, cs, _ = c.pack(x)
        v = 0.3 * torch.randn_like(x)
        out = []
        for f in (lambda: c.pack(x), lambda: c.kick_drift(pos, cs, v, v, 0.1, 0.5)):
            best = float("inf")
            for _ in range(5):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                for _ in range(20):
                    f()
                b.record()
                torch.cuda.synchronize()
                best = min(best, a.elapsed_time(b))
            out.append(best)
        return out

    with_it, without = time(7000), time(0)
    assert all(a <= 1.8 * b for a, b in zip(with_it, without)), (with_it, without)
