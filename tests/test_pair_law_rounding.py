"""The rounding error of the FP32 pair law over whole distributions of separations, on
the host with the kernels' own operations, against eqs. 2 and 4d in x87 extended
precision.

Two figures per softening: the rms of the error of g r relative to the rms of g r for
separations uniform in the sphere of the cutoff (what enters a particle's force), and the
rms of q times the relative error for q = 1 - r/b_f log-uniform in [5e-4, 0.1] (what the
rounding of s leaves near the cutoff).  The bounds are those of a law without a fifth
root, g = h(s) (1 - s/b_f^2)^4 with cubic rows, which rounds its fastest-growing factor
four times: its own figures, and 2% on the second, which s alone decides."""
import numpy as np
import pytest

X = np.longdouble

# b_f, b_pp, and the figures of that law
LAWS = [(2.0, 0.2, 1.23e-7, 6.33e-8), (1.5, 0.1, 1.56e-7, 1.14e-7), (1.0, 0.3, 1.14e-7, 6.29e-8),
        (3.0, 0.3, 1.16e-7, 1.14e-7), (3.5, 0.0625, 3.57e-7, 1.70e-7)]


def _poly(c, t):
    s = np.zeros_like(t)
    for v in reversed(c):
        s = s * t + X(v)
    return s


def _r_over_r(r, b):
    t = r / b
    p1 = _poly([X(64) / 5, 0, -X(256) / 5, 32, X(1536) / 35, -X(192) / 5], t)
    p2 = _poly([X(256) / 5, -96, X(256) / 5, 32, -X(1536) / 35, X(64) / 5], t) + X(3) / 35 / t ** 3 - X(32) / 5 / t
    return np.where(t < 0.5, p1, np.where(t < 1, p2, t ** -3)) / b ** 3


def _g(r, b_pp, b_f):
    q = 1 - r / b_f
    tail = q ** 5 * _poly([X(1344) / 35, -X(2912) / 35, X(2048) / 35, -X(64) / 5], q) / r ** 3
    return np.where((r >= b_pp) & (2 * r >= b_f), tail, _r_over_r(r, b_pp) - _r_over_r(r, b_f))


@pytest.mark.parametrize("b_f,b_pp,weighted,near", LAWS)
def test_error_of_the_law(b_f, b_pp, weighted, near):
    import paper_2512_12629_amd as m
    h = m.cube2_create(m.Config(n_fine=64, b_fine=b_f, b_pp=b_pp).c())
    try:
        rng = np.random.default_rng(5)
        n = 400000
        for r in (b_f * rng.random(n) ** (1 / 3), b_f * (1 - np.exp(rng.uniform(np.log(5e-4), np.log(0.1), n)))):
            u = rng.standard_normal((3, n))
            d = (np.rint(u / np.linalg.norm(u, axis=0) * r * 2 ** 15) * 2.0 ** -15).astype(np.float32)
            rr = np.sqrt((d.astype(X) ** 2).sum(axis=0))
            keep = (rr > 0) & (rr < b_f * 0.9995)
            d, rr = np.ascontiguousarray(d[:, keep]), rr[keep]
            ref = _g(rr, X(b_pp), X(b_f))
            for got in (m.cube2_pair_law_f32(h, d), m.cube2_pair_jacobian_f32(h, d)[0]):
                e = got.astype(X) - ref
                if r.min() < 0.8 * b_f:
                    assert np.sqrt(((e * rr) ** 2).sum() / ((ref * rr) ** 2).sum()) <= weighted
                else:
                    assert np.sqrt(((e / ref * (1 - rr / b_f)) ** 2).mean()) <= 1.02 * near
    finally:
        m.cube2_destroy(h)
