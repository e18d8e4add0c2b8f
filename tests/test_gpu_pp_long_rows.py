"""The PP force where one x-row of cells holds thousands of particles: a core of strong
pairs and an edge of weak ones near the cutoff, which a plain FP32 sum over the row
loses.  The rms error against the oracle is at most 1.5e-7 of the rms force: the law's own
0.9e-7 and, of ranges of 512 terms over four lanes, 2.4e-8 sqrt(128 / 3) / 2 = 8e-8 of one
range, a twelfth of the sum each."""
import numpy as np
import pytest

import oracle
from helpers import ios_decode

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("core,edge", [(3000, 3000), (1500, 4500), (600, 2000)])
def test_core_and_edge_in_one_row(core, edge):
    import paper_2512_12629_amd as m
    rng = np.random.default_rng(core + edge)
    x = np.concatenate([np.array([[20.3], [20.5], [20.5]]) + 0.1 * rng.standard_normal((3, core)),
                        np.array([[22.15], [20.5], [20.5]]) + 0.08 * rng.standard_normal((3, edge)),
                        64.0 * rng.random((3, 3000))], axis=1) / 64.0
    x = np.ascontiguousarray(x).astype(np.float32)
    c = m.Cube2(m.Config(n_fine=64), n_max=x.shape[1])
    pos, cs, _ = c.pack(torch.from_numpy(x).cuda())
    xf = ios_decode(pos.cpu().numpy().view(np.uint16), cs.cpu().numpy().view(np.uint32), 64) / 2.0 ** 15
    ref = oracle.Oracle(oracle.Params(n_fine=64, coarse_ratio=0)).pp_accel(xf)
    e = c.pp_force(pos, cs).double().cpu().numpy() - ref
    assert np.sqrt((e ** 2).mean() / (ref ** 2).mean()) <= 1.5e-7
