"""The PP kernels at numbers of light tiles that are no multiple of the 8 XCDs and lie at
the steps of the claims' size (strides or counters, chunks of 2, 3 and 4 items): every
light tile's pair sums are formed once.

An output that holds NaN before shows sums that were left out, one that is added to shows
sums that were added twice; the force and its adjoint, whose PP runs on a part of the
grid, equal their separate parts bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _state(n_fine, light):
    """A mesh with `light` light tiles: a dense cell in the middle of each of the others."""
    import paper_2512_12629_amd as m
    nt = n_fine // 16
    rng = np.random.default_rng(light)
    t = rng.permutation(nt ** 3)[:nt ** 3 - light]
    at = 16.0 * np.stack([t % nt, t // nt % nt, t // nt ** 2]) + 8.0
    x = np.concatenate([np.repeat(at, 540, axis=1) + 1.9 * rng.random((3, 540 * t.size)),
                        (n_fine - 0.1) * rng.random((3, 5 * nt ** 3))], axis=1) / n_fine
    x = torch.from_numpy(np.ascontiguousarray(x).astype(np.float32)).cuda()
    c = m.Cube2(m.Config(n_fine=n_fine), n_max=x.shape[1])
    pos, cs, _ = c.pack(x)
    c.work.fill_(255)       # scratch left by an earlier call: NaN
    g = torch.Generator(device="cuda").manual_seed(light)
    return m, c, pos, cs, torch.randn(x.shape, generator=g, device="cuda")


@pytest.mark.parametrize("light", [2308, 3452, 4093])
def test_adjoint_alone(light):
    m, c, pos, cs, ab = _state(256, light)
    plain = torch.full_like(ab, float("nan"))
    m.cube2_pp_force_backward(c.ctx, pos, cs, ab, plain, c.work)
    assert not plain.isnan().any()
    assert torch.equal(c.pp_force_backward(pos, cs, ab, x_bar=ab.clone()), ab + plain)


@pytest.mark.parametrize("light", [1444, 2156, 2876])
def test_adjoint_beside_pm(light):
    m, c, pos, cs, ab = _state(256, light)
    whole = c.force_backward(pos, cs, ab)
    parts = c.pp_force_backward(pos, cs, ab, x_bar=c.pm_force_backward(pos, cs, ab))
    assert torch.equal(whole, parts)


@pytest.mark.parametrize("light", [4100, 6140, 8190])
def test_force_alone(light):
    m, c, pos, cs, a0 = _state(512, light)
    plain = torch.full_like(a0, float("nan"))
    m.cube2_pp_force(c.ctx, pos, cs, plain, c.work)
    assert not plain.isnan().any()
    assert torch.equal(c.pp_force(pos, cs, acc=a0.clone()), a0 + plain)
    none = torch.zeros(32 ** 3, dtype=torch.uint8, device="cuda")
    skipped = a0.clone()
    m.cube2_pp_force_skip(c.ctx, pos, cs, none, skipped, c.work, accumulate=True)
    assert torch.equal(skipped, a0 + plain)


@pytest.mark.parametrize("n_fine,light", [(256, 3076), (512, 4604), (512, 6143)])
def test_force_beside_pm(n_fine, light):
    m, c, pos, cs, _ = _state(n_fine, light)
    whole = c.force(pos, cs)
    assert torch.equal(whole, c.pp_force(pos, cs, acc=c.pm_force(pos, cs)))
