"""Interpolation with a coarse level of ratio 2, as the lines of the coarse potential (up to
2048 particles per tile) and as its node forces (more): both levels, the coarse level
alone and the FP64 form against the oracle, at the bars of their other tests.  And with few
particles per tile ratio 2 must not cost much more than ratio 4."""
import numpy as np
import pytest

import oracle
from helpers import force_stats, ios_decode

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("assign", ["cic", "tsc"])
@pytest.mark.parametrize("n_fine,n", [(16, 2048), (16, 2049), (32, 1), (32, 16384), (32, 16385), (128, 4000)])
def test_either_side_of_the_limit(n_fine, n, assign):
    import paper_2512_12629_amd as m
    rng = np.random.default_rng(n)
    p = 3 if assign == "tsc" else 2
    x = torch.from_numpy(rng.random((3, n)).astype(np.float32) * np.float32(0.9999)).cuda()
    flags = m.CUBE2_FP64_FORM | (m.CUBE2_ASSIGN_TSC if p == 3 else 0)
    try:
        c = m.Cube2(m.Config(n_fine=n_fine, coarse_ratio=2, flags=flags), n_max=n)
    except m.Cube2Error:
        pytest.skip("the coarse mesh is too small")
    pos, cs, _ = c.pack(x)
    xf = ios_decode(pos.cpu().numpy().view(np.uint16), cs.cpu().numpy().view(np.uint32), n_fine) / 2.0 ** 15
    phis = [torch.from_numpy(rng.standard_normal((k, k, k)).astype(np.float32)).cuda()
            for k in (n_fine, n_fine // 2)]
    got = c.interp(pos, cs, *phis).cpu().numpy().astype(np.float64)
    ref = sum(oracle.interp(xf, oracle.fd_force(f.cpu().numpy().astype(np.float64)), H, True, p) / H ** 2
              for f, H in zip(phis, (1, 2)))
    med, p99, _ = force_stats(got, ref)
    assert med < 1e-5 and p99 < 1e-4, (med, p99)
    if n == 1:
        return    # its own mesh force is zero but for rounding
    o = oracle.Oracle(oracle.Params(n_fine=n_fine, coarse_ratio=2, assign=p))
    med, p99, _ = force_stats(c.pm_force_f64(pos, cs).cpu().numpy(), o.pm_accel(xf))
    assert med < 1e-10 and p99 < 1e-8, (med, p99)
    med, p99, _ = force_stats(c.pm_level_force(pos, cs, 1).cpu().numpy(), o.pm_level_accel(xf, 0))
    assert med < 1e-4 and p99 < 1e-3, (med, p99)


def test_ratio_two_costs_little_more_than_ratio_four():
    import paper_2512_12629_amd as m
    n = 153 ** 3
    x = torch.from_numpy(np.random.default_rng(1).random((3, n)).astype(np.float32) * np.float32(0.9999)).cuda()

    def time(ratio):
        c = m.Cube2(m.Config(n_fine=512, coarse_ratio=ratio), n_max=n)
        pos, cs, _ = c.pack(x)
        phis = [torch.randn((k, k, k), device="cuda") for k in (512, 512 // ratio)]
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                c.interp(pos, cs, *phis)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    assert time(2) <= 1.25 * time(4)
