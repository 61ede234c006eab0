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
    for _ in range(20):                    # more than the sets of scratch
        S.dt.zero_()
        gbr.gbr_compute_dt(S.ctx, S.Q, P.cfl, S.dt, S.stream)
        torch.cuda.synchronize()
        assert float(S.dt.cpu()[0]) == want
    assert S.check() == gbr.GBR_OK
    S.close()


def test_calls_of_one_context_that_overlap():
    """Eight calls of one context, each on its own stream and its own state."""
    from paper_2305_00762_amd.solver import Solver
    torch = require_gpu()
    ps = [PB.riemann(96, seed=20 + k) for k in range(8)]
    want = [O.dt(ocfg(P), P.Q, P.cfl) for P in ps]
    S = Solver(ps[0])
    Q = [torch.from_numpy(P.Q.copy()).cuda() for P in ps]
    dt = torch.zeros(8, dtype=torch.float64, device="cuda")
    streams = [torch.cuda.Stream() for _ in ps]
    torch.cuda.synchronize()
    for _ in range(10):
        dt.zero_()
        torch.cuda.synchronize()
        for k, s in enumerate(streams):
            gbr.gbr_compute_dt(S.ctx, Q[k], ps[k].cfl, dt[k:k + 1], s)
        torch.cuda.synchronize()
        assert dt.cpu().tolist() == want
    S.close()
