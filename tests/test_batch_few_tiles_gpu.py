"""Batches on both sides of the number of 15x15 tiles below which the two 15x15
forms give a lane two interfaces instead of four: inviscid and viscous grids, ragged
edges, both precisions.  Bars: each grid as its single-grid run, 1e-12 norm-wise
relative, state and time step (the batch tests' bar); FP64 states the oracle's."""
import numpy as np
import pytest

import oracle as O
from paper_2305_00762_amd import gbr
from paper_2305_00762_amd import problems as PB
from gpu_util import ocfg, relerr, require_gpu
from test_batch_gpu import single_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [gbr.GBR_PREC_FP64, gbr.GBR_PREC_FP32_BULK])
@pytest.mark.parametrize("form", [1, 3])
@pytest.mark.parametrize("tiles", [1, 40, 2199, 2200])
def test_both_sides_of_the_line(tiles, form, precision):
    from paper_2305_00762_amd.solver import BatchSolver
    torch = require_gpu()
    big = {2199: (9, 242), 2200: (10, 218)}.get(tiles)       # + 21 or 20 tiles of small grids
    if tiles == 1:
        ps = [PB.riemann(14, seed=1, ny=13)]
    else:
        ps = [PB.riemann(43, seed=1, ny=40), PB.shear(31, seed=2, ny=33)]        # 9 + 9
        if tiles == 40:
            ps += [PB.riemann(70, seed=3, ny=50), PB.vortex(14)]                 # 20 + 1
            ps += [PB.free_stream(15, ny=12)]                                    # 1
        else:
            ps += [PB.riemann(15 * big[0] - 3, seed=3, ny=15 * big[1] - 7)]
            ps += [PB.vortex(30, ny=15)]                                         # 2
            if tiles == 2199:
                ps += [PB.free_stream(15, ny=12)]                                # 1
    B = BatchSolver(ps, precision=precision)
    gbr.gbr_batch_set_tiling(B.b, form)
    assert gbr.gbr_batch_info(B.b)[3] == tiles
    dts = []
    for _ in range(2):
        B.step()
        dts.append(B.dt())
    torch.cuda.synchronize()
    assert B.check() == gbr.GBR_OK
    for k, P in enumerate(ps):
        got = B.states()[k].cpu().numpy()
        ref, ref_dt = single_run(P, precision, 1, 2)
        assert relerr(got, ref.cpu().numpy()).max() <= 1e-12
        assert np.abs(np.array([d[k] for d in dts]) - ref_dt).max() <= 1e-12 * max(ref_dt)
        if precision == gbr.GBR_PREC_FP64 and P.nx * P.ny < 10000:
            Q = P.Q.copy()
            for _ in range(2):
                O.step(ocfg(P), Q, P.cfl)
            assert relerr(got, Q).max() <= 1e-12
    B.close()
