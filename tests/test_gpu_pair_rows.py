"""The FP32 pair-law tables, which the device makes in cube2_init_tables, equal the rows
that the host evaluators form: 32768 isolated pairs, their separations spread over every
octave of the table and the cutoff, get g(D) D with the host's g, bit for bit (G m = 1),
with the cutoff inside a row and at an edge of one, clamped and not, both reaches.  And
making a context is cheap."""
import time

import numpy as np
import pytest

from helpers import ios_decode


@pytest.mark.gpu
@pytest.mark.parametrize("b_f,b_pp", [(2.0, 0.2), (1.5, 0.1), (1.0, 0.3), (2.0, 0.03125), (0.25, 0.00390625),
                                      (3.5, 0.0625), (3.0, 0.046875)])
def test_isolated_pairs_bit_for_bit(b_f, b_pp):
    torch = pytest.importorskip("torch")
    import paper_2512_12629_amd as m
    rng = np.random.default_rng(2)
    n = 32 ** 3
    k = np.stack(np.meshgrid(*[np.arange(32)] * 3, indexing="ij")).reshape(3, -1)
    r = np.concatenate([np.exp(rng.uniform(np.log(2.0 ** -14), np.log(1.1 * b_f), n // 2)),
                        b_f * rng.random(n // 4) ** (1 / 3), b_f * (1 - 10 ** rng.uniform(-5, -1, n // 4))])
    u = rng.standard_normal((3, n))
    d = np.rint(u / np.linalg.norm(u, axis=0) * r * 2 ** 15).astype(np.int64)
    a = (k << 18) + (1 << 17)                                     # one pair per 8^3 fine cells
    q = np.concatenate([a, a + d], axis=1)
    x = ((q + 0.5) / (256 << 15))
    c = m.Cube2(m.Config(n_fine=256, b_fine=b_f, b_pp=b_pp), n_max=2 * n)
    pos, cs, perm = c.pack(torch.from_numpy(np.ascontiguousarray(x.astype(np.float32))).cuda())
    perm = perm.cpu().numpy()
    qs = np.empty((3, 2 * n), np.int64)
    qs[:, perm] = ios_decode(pos.cpu().numpy().view(np.uint16), cs.cpu().numpy().view(np.uint32), 256)
    got = np.empty((3, 2 * n), np.float32)
    got[:, perm] = c.pp_force(pos, cs).cpu().numpy()
    dj = np.ascontiguousarray(((qs[:, n:] - qs[:, :n]) * 2.0 ** -15).astype(np.float32))
    g = m.cube2_pair_law_f32(c.ctx, dj)
    want = g * dj
    # (below 1e-30 the kernel's scaled sum may be subnormal; a second particle of a pair
    # longer than 2 may meet that of the next pair)
    normal = np.abs(want) >= 1e-30
    assert np.array_equal(got[:, :n][normal], want[normal])
    if b_f <= 2.0:
        assert np.array_equal(got[:, n:][normal], -want[normal])
    assert np.all(np.abs(got[:, :n][~normal]) < 1.1e-30)


def test_context_is_cheap_to_make():
    """5 to 17 us; 350 to 430 when the host made the FP32 tables for every context."""
    import paper_2512_12629_amd as m
    best = float("inf")
    for _ in range(200):
        t = time.perf_counter()
        h = m.cube2_create(m.Config(n_fine=64).c())
        best = min(best, time.perf_counter() - t)
        m.cube2_destroy(h)
    assert best < 100e-6
