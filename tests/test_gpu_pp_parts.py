"""The PP kernels' list of parts (heavy tiles with much work, split): boxes of a uniform
density around the light tiles' limit and far above it, for both reaches, and more parts
than the list holds, against the oracle for the force and its adjoint (median 1e-4, p99
1e-3 relative to max(|F|, 1e-6 median |F|)); and that a box is not slower for holding
fewer particles, just above the limit, where parts would not pay."""
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


@pytest.mark.parametrize("b_fine,b_pp", [(2.0, 0.2), (3.5, 0.0625)])
@pytest.mark.parametrize("side", [34, 38, 64])
def test_uniform(side, b_fine, b_pp):
    _check(np.random.default_rng(side).random((3, side ** 3)), 64, b_fine, b_pp)


def test_more_parts_than_the_list_holds():
    """300 tiles that make 32 parts each: 3400 particles and a dense cell of 700."""
    rng = np.random.default_rng(8)
    t = rng.permutation(4096)[:300]
    at = 16.0 * np.stack([t % 16, t // 16 % 16, t // 256])
    x = np.concatenate([np.repeat(at, 3400, axis=1) + 15.9 * rng.random((3, 3400 * 300)),
                        np.repeat(at + 8.0, 700, axis=1) + 1.9 * rng.random((3, 700 * 300)),
                        255.9 * rng.random((3, 20000))], axis=1)
    _check(x / 256.0, 256)


def _pp_time(side, n_fine):
    import paper_2512_12629_amd as m
    g = torch.Generator(device="cuda").manual_seed(side)
    k = torch.arange(side, device="cuda") + 0.5
    x = torch.stack(torch.meshgrid(k, k, k, indexing="ij")).reshape(3, -1)
    x = (x + 0.15 * torch.randn(x.shape, generator=g, device="cuda")) / side % 1.0
    c = m.Cube2(m.Config(n_fine=n_fine), n_max=x.shape[1])
    pos, cs, _ = c.pack(x.contiguous())
    out = torch.empty_like(x)
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            m.cube2_pp_force(c.ctx, pos, cs, out, c.work)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def test_fewer_particles_are_not_slower():
    assert _pp_time(135, 256) <= 1.3 * _pp_time(144, 256)
