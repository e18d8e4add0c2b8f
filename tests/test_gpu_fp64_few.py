"""The FP64 PP force where tiles hold only a few particles (one wave reads its neighbours
from memory) with dense tiles between them: particles whose neighbours are the same get
the same force, by either kernel, as when the rest of the box is full (FP64 rounding,
1e-11 of the force and its median); against the oracle as the FP64 form's other tests."""
import numpy as np
import pytest

import oracle
from helpers import ios_decode

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
N_FINE = 256


def _low(rng, cells):
    """5000 particles below z = 112 and cells[i] more in one IOS cell of tiles along x."""
    x = [np.array([[255.9], [255.9], [103.0]]) * rng.random((3, 5000)) + np.array([[0.0], [0.0], [9.0]])]
    for i, k in enumerate(cells):
        x.append(np.array([[30.0 + 32 * i], [46.0], [62.0]]) + 1.99 * rng.random((3, k)))
    return np.concatenate(x, axis=1)


def _force(x, b_fine, b_pp):
    import paper_2512_12629_amd as m
    x = np.ascontiguousarray(x / N_FINE).astype(np.float32)
    c = m.Cube2(m.Config(n_fine=N_FINE, b_fine=b_fine, b_pp=b_pp, flags=m.CUBE2_FP64_FORM), n_max=x.shape[1])
    pos, cs, perm = c.pack(torch.from_numpy(x).cuda())
    f = c.pp_force_f64(pos, cs)
    assert torch.equal(c.pp_force_f64(pos, cs, f.clone()), f + f)
    q = ios_decode(pos.cpu().numpy().view(np.uint16), cs.cpu().numpy().view(np.uint32), N_FINE)
    return f.cpu().numpy(), perm.cpu().numpy(), q / 2.0 ** 15


@pytest.mark.parametrize("b_fine,b_pp", [(2.0, 0.2), (3.5, 0.0625)])
@pytest.mark.parametrize("cells", [(), (1, 2, 63, 64, 65), (127, 128, 129, 400)])
def test_as_in_a_full_box(cells, b_fine, b_pp):
    rng = np.random.default_rng(len(cells))
    low = _low(rng, cells)
    n = low.shape[1]
    f, perm, xf = _force(low, b_fine, b_pp)
    ref = oracle.Oracle(oracle.Params(n_fine=N_FINE, b_fine=b_fine, b_pp=b_pp)).pp_accel(xf)
    r = np.linalg.norm(ref, axis=0)
    e = np.linalg.norm(f - ref, axis=0)[r > 0] / np.maximum(r[r > 0], 1e-6 * np.median(r[r > 0]))
    assert np.median(e) < 1e-9 and np.percentile(e, 99) < 1e-5
    # more than 64 particles per tile: the other kernel for all
    top = np.array([[255.9], [255.9], [111.0]]) * rng.random((3, 64 * 16 ** 3)) + np.array([[0.0], [0.0], [136.0]])
    g, perm2, _ = _force(np.concatenate([low, top], axis=1), b_fine, b_pp)
    assert np.array_equal(perm2[:n], perm)
    g = g[:, :n]
    r = np.linalg.norm(g, axis=0)
    assert np.all(f[:, r == 0] == 0)
    assert np.all(np.linalg.norm(f - g, axis=0) <= 1e-11 * (r + np.median(r[r > 0])))


@pytest.mark.parametrize("n", [0, 1, 64 * 16 ** 3, 64 * 16 ** 3 + 1])
def test_sizes_at_the_limit(n):
    import paper_2512_12629_amd as m
    x = np.random.default_rng(n).random((3, n)).astype(np.float32) * np.float32(0.9999)
    c = m.Cube2(m.Config(n_fine=N_FINE, flags=m.CUBE2_FP64_FORM), n_max=max(n, 1))
    pos, cs, _ = c.pack(torch.from_numpy(x).cuda())
    f = c.pp_force_f64(pos, cs)
    if n > 1:
        xf = ios_decode(pos.cpu().numpy().view(np.uint16), cs.cpu().numpy().view(np.uint32), N_FINE) / 2.0 ** 15
        idx = np.arange(0, n, 97)
        ref = oracle.Oracle(oracle.Params(n_fine=N_FINE)).pp_accel_subset(xf, idx)
        r = np.linalg.norm(ref, axis=0)
        e = np.linalg.norm(f.cpu().numpy()[:, idx] - ref, axis=0)[r > 0] / np.maximum(r[r > 0], 1e-6 * np.median(r[r > 0]))
        assert np.median(e) < 1e-9 and np.percentile(e, 99) < 1e-5
    else:
        assert torch.all(f == 0)


def test_few_particles_cost_little():
    import paper_2512_12629_amd as m

    def time(n):
        x = torch.from_numpy(np.random.default_rng(1).random((3, n)).astype(np.float32) * np.float32(0.9999)).cuda()
        c = m.Cube2(m.Config(n_fine=N_FINE, flags=m.CUBE2_FP64_FORM), n_max=n)
        pos, cs, _ = c.pack(x)
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                c.pp_force_f64(pos, cs)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    assert time(38 ** 3) <= 0.45 * time(76 ** 3)
