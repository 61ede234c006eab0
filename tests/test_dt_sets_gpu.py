"""The time step of a state and that of stage-3 extrema on one context, in turn
and at the same time, over every tile shape (each leaves another number of
extrema): bit for bit the values of calls made one by one."""
import pytest

from paper_2305_00762_amd import gbr
from paper_2305_00762_amd import problems as PB
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


def stage3(S):
    gbr.gbr_rk_stage(S.ctx, 3, S.dt, S.Q, S.Q, S.Q1, S.stream)


@pytest.mark.parametrize("mu", [0.0, 1e-3])
@pytest.mark.parametrize("n", [12, 90, 400])
def test_extrema_of_every_shape(n, mu):
    from paper_2305_00762_amd.solver import Solver
    torch = require_gpu()
    P = PB.riemann(n, seed=5, ny=n + 7)
    P.mu = mu
    S = Solver(P)
    S.compute_dt()
    a, b = torch.zeros_like(S.dt), torch.zeros_like(S.dt)
    for k in range(20):
        gbr.gbr_set_tiling(S.ctx, k % 4)
        stage3(S)
        for _ in range(k % 3):
            gbr.gbr_compute_dt(S.ctx, S.Q1, P.cfl, b, S.stream)
        gbr.gbr_stage_dt(S.ctx, P.cfl, a, S.stream)
        gbr.gbr_compute_dt(S.ctx, S.Q1, P.cfl, b, S.stream)
        torch.cuda.synchronize()
        assert float(a) == float(b) > 0.0
    assert S.check() == gbr.GBR_OK
    S.close()


@pytest.mark.parametrize("n,calls", [(64, 8), (2048, 1)])
def test_both_kinds_at_the_same_time(n, calls):
    """Eight calls on a small grid (one launch each), one of two launches on a
    grid of 4M cells, beside a call on stage-3 extrema."""
    from paper_2305_00762_amd.solver import Solver
    torch = require_gpu()
    S = Solver(PB.riemann(n, seed=6))
    cfl = S.p.cfl
    Q = [torch.from_numpy(PB.riemann(n, seed=30 + k).Q).cuda() for k in range(calls)]
    dt = torch.zeros(calls + 1, dtype=torch.float64, device="cuda")
    S.compute_dt()
    stage3(S)
    gbr.gbr_stage_dt(S.ctx, cfl, dt[:1])
    for k, q in enumerate(Q):
        gbr.gbr_compute_dt(S.ctx, q, cfl, dt[k + 1:k + 2])
    torch.cuda.synchronize()
    want = dt.cpu().tolist()
    assert min(want) > 0.0 and len(set(want)) == calls + 1
    streams = [torch.cuda.Stream() for _ in range(calls + 1)]
    for _ in range(10):
        dt.zero_()
        stage3(S)
        torch.cuda.synchronize()
        for k, s in enumerate(streams):
            if k == 0:
                gbr.gbr_stage_dt(S.ctx, cfl, dt[:1], s)
            else:
                gbr.gbr_compute_dt(S.ctx, Q[k - 1], cfl, dt[k:k + 1], s)
        torch.cuda.synchronize()
        assert dt.cpu().tolist() == want
    S.close()
