"""The time step in one launch (small grids) and in two, on both sides of the
line and with repeated calls on one context: bit for bit the oracle's."""
import pytest

import oracle as O
from paper_2305_00762_amd import gbr
from paper_2305_00762_amd import problems as PB
from gpu_util import ocfg, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mu", [0.0, 1e-3])
@pytest.mark.parametrize("nx,ny", [(12, 12), (16, 16), (17, 16), (64, 64), (128, 128), (200, 200),
                                   (201, 200)])
def test_dt_bit_exact_and_repeatable(nx, ny, mu):
    from paper_2305_00762_amd.solver import Solver
    torch = require_gpu()
    P = PB.riemann(nx, seed=8, ny=ny)
    P.mu = mu
    want = O.dt(ocfg(P), P.Q, P.cfl)
    S = Solver(P)
    for _ in range(5):
        S.dt.zero_()
        gbr.gbr_compute_dt(S.ctx, S.Q, P.cfl, S.dt, S.stream)
        torch.cuda.synchronize()
        assert float(S.dt.cpu()[0]) == want
    assert S.check() == gbr.GBR_OK
    S.close()
