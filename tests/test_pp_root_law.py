"""The FP32 pair law's table at its edges: configurations whose octaves from
the smallest tabulated s to the largest of the staged box exceed the table
(s is then clamped to the first row beyond the cutoff), boxes that pass
through LDS in parts with both neighbour reaches, and tiles split in parts.

The law on the host against the exact rational law, with the bound of the
other pins, |g32 - g| <= (2e-6 + 1e-6/q) |g|, q = 1 - r/b_f; the kernels
against the oracle with the bar of the other PP tests (median 1e-4, p99 1e-3
relative to max(|F|, 1e-6 median |F|))."""
from fractions import Fraction as Fr

import numpy as np
import pytest

import oracle
from helpers import ios_decode
from oracle import exact

torch = pytest.importorskip("torch")

CLAMPED = [(2.0, 0.03125), (0.25, 0.00390625), (3.0, 0.046875), (0.5, 0.05)]


@pytest.mark.parametrize("b_f,b_pp", CLAMPED)
def test_clamped_law_against_exact_rational(b_f, b_pp):
    import paper_2512_12629_amd as m
    h = m.cube2_create(m.Config(n_fine=64, b_fine=b_f, b_pp=b_pp).c())
    try:
        rng = np.random.default_rng(17)
        r = np.concatenate([np.exp(rng.uniform(np.log(2.0 ** -14), np.log(1.2 * b_f), 200)),
                            b_f * (1 + np.array([-1e-3, -1e-4, 0.0, 1e-4])),
                            rng.uniform(b_f, 3.4 if b_f <= 2 else 5.1, 40)])
        u = rng.standard_normal((3, r.size))
        u /= np.linalg.norm(u, axis=0)
        n = np.rint(u * r * 2 ** 15).astype(np.int64)
        n[:, 0] = 0
        d = (n * 2.0 ** -15).astype(np.float32)
        g32 = m.cube2_pair_law_f32(h, d).astype(np.float64)
        ga = m.cube2_pair_jacobian_f32(h, d)[0].astype(np.float64)
        assert np.isfinite(g32[0]) and np.isfinite(ga[0])
        bpp, bf = Fr(b_pp).limit_denominator(10 ** 12), Fr(b_f).limit_denominator(10 ** 12)
        for i in range(1, n.shape[1]):
            n2 = int((n[:, i] ** 2).sum())
            q = 1.0 - (n2 * 2.0 ** -30) ** 0.5 / b_f
            for v in (g32[i], ga[i]):
                if q <= 0:
                    assert v == 0.0
                else:
                    g = float(exact.pair_g(n2, bpp, bf))
                    assert abs(v - g) <= (2e-6 + 1e-6 / q) * abs(g), (i, n[:, i], v, g)
    finally:
        m.cube2_destroy(h)


def _rel(got, ref):
    fr = np.linalg.norm(ref, axis=0)
    has = fr > 0
    e = np.linalg.norm(got - ref, axis=0)[has] / np.maximum(fr[has], 1e-6 * np.median(fr[has]))
    return float(np.median(e)), float(np.percentile(e, 99))


# (b_f, b_pp, particles in the column): one that is staged at once, one that
# passes through LDS in parts, for both reaches, clamped and not
@pytest.mark.gpu
@pytest.mark.parametrize("b_f,b_pp,n_col", [(2.0, 0.03125, 1500), (2.0, 0.03125, 5200),
                                            (3.0, 0.046875, 1500), (3.0, 0.046875, 5200),
                                            (3.5, 0.0625, 5200), (1.5, 0.1, 5200)])
def test_pp_and_adjoint_against_oracle(b_f, b_pp, n_col):
    import paper_2512_12629_amd as m
    n_fine = 64
    rng = np.random.default_rng(n_col)
    bg = rng.random((3, 3000))
    col = (np.array([[20.0], [20.0], [16.0]]) + np.array([[4.0], [4.0], [16.0]]) * rng.random((3, n_col))) / n_fine
    x = np.ascontiguousarray(rng.permutation(np.concatenate([bg, col], axis=1).T).T).astype(np.float32)
    c = m.Cube2(m.Config(n_fine=n_fine, coarse_ratio=4, b_fine=b_f, b_pp=b_pp), n_max=x.shape[1])
    pos, cs, _ = c.pack(torch.from_numpy(x).cuda())
    q = ios_decode(pos.cpu().numpy().view(np.uint16), cs.cpu().numpy().view(np.uint32), n_fine)
    xf = q / 2.0 ** 15
    o = oracle.Oracle(oracle.Params(n_fine=n_fine, coarse_ratio=4, b_fine=b_f, b_pp=b_pp))
    abar = rng.standard_normal(x.shape).astype(np.float32)
    med, p99 = _rel(c.pp_force(pos, cs).double().cpu().numpy(), o.pp_accel(xf))
    assert med < 1e-4 and p99 < 1e-3, (med, p99)
    xb = c.pp_force_backward(pos, cs, torch.from_numpy(abar).cuda()).double().cpu().numpy()
    med, p99 = _rel(xb, o.pp_adjoint(xf, abar.astype(np.float64)))
    assert med < 1e-4 and p99 < 1e-3, (med, p99)
