"""The adjoint of the mass assignment, each level, each assignment, with few tiles and many
and with few and many particles in each, against the oracle's (median 1e-5, p99 1e-4 as
its other tests).  And the coarse level's must not cost more than the fine level's, whose
mesh is many times larger."""
import numpy as np
import pytest

import oracle
from helpers import force_stats, ios_decode

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("assign", ["cic", "tsc"])
@pytest.mark.parametrize("n_fine,ratio,n", [(32, 2, 3), (32, 2, 20000), (64, 8, 5000), (256, 2, 1),
                                            (256, 4, 30000), (256, 8, 2048 * 4096 + 1)])
def test_against_oracle(n_fine, ratio, n, assign):
    import paper_2512_12629_amd as m
    rng = np.random.default_rng(n)
    p = 3 if assign == "tsc" else 2
    x = torch.from_numpy(rng.random((3, n)).astype(np.float32) * np.float32(0.9999)).cuda()
    c = m.Cube2(m.Config(n_fine=n_fine, coarse_ratio=ratio, flags=m.CUBE2_ASSIGN_TSC if p == 3 else 0), n_max=n)
    pos, cs, _ = c.pack(x)
    xf = ios_decode(pos.cpu().numpy().view(np.uint16), cs.cpu().numpy().view(np.uint32), n_fine) / 2.0 ** 15
    o = oracle.Oracle(oracle.Params(n_fine=n_fine, coarse_ratio=ratio, assign=p))
    for level, k in ((0, n_fine), (1, n_fine // ratio)):
        rb = rng.standard_normal((k, k, k)).astype(np.float32)
        got = c.deposit_backward(pos, cs, torch.from_numpy(rb).cuda(), level).cpu().numpy()
        ref = o.deposit_adjoint(xf, rb.astype(np.float64), level=1 - level)
        med, p99, _ = force_stats(got, ref)
        assert med < 1e-5 and p99 < 1e-4, (level, med, p99)


@pytest.mark.parametrize("assign", ["cic", "tsc"])
def test_coarse_level_costs_no_more_than_the_fine(assign):
    import paper_2512_12629_amd as m
    n = 128 ** 3
    x = torch.from_numpy(np.random.default_rng(1).random((3, n)).astype(np.float32) * np.float32(0.9999)).cuda()
    c = m.Cube2(m.Config(n_fine=256, coarse_ratio=2, flags=m.CUBE2_ASSIGN_TSC if assign == "tsc" else 0), n_max=n)
    pos, cs, _ = c.pack(x)

    def time(level, k):
        rb = torch.randn((k, k, k), device="cuda")
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                c.deposit_backward(pos, cs, rb, level)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    assert time(1, 128) <= 1.3 * time(0, 256)
