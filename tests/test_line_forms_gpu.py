"""The line-streamed stage kernel in every launch form: interfaces per lane
chosen by the number of tiles (both sides of the rule, on grids whose last tiles
are ragged), every tile shape, the schemes that instantiate it.

Bars: detector flags bit for bit; a residual within 1e-12 (FP64) or 1e-6 (FP32
bulk) of the flux-divergence scale max|F|/dx, the bars the other residual tests
derive.  The noise field flags almost every interface, so each wave's queue of
flagged interfaces overflows one round of 64 several times."""
import numpy as np
import pytest

import oracle as O
from paper_2305_00762_amd import gbr
from paper_2305_00762_amd import problems as PB
from gpu_util import ocfg, report, require_gpu, res_err

pytestmark = pytest.mark.gpu


def noise(nx, ny, mu, bc):
    rng = np.random.default_rng(nx * 1000 + ny)
    rho, p = rng.uniform(0.5, 1.5, (2, ny, nx))
    u, v = rng.uniform(-0.5, 0.5, (2, ny, nx))
    P = PB.free_stream(nx, ny=ny, bc=bc)
    P.Q = PB.prim_to_state(rho, u, v, p)
    P.mu = mu
    return P


def check(name, P, tiling, precision=0, recon=0, order=7, riemann=0):
    from paper_2305_00762_amd.solver import Solver
    torch = require_gpu()
    P.riemann = riemann
    S = Solver(P, export_flags=True, precision=precision, recon=recon, order=order)
    gbr.gbr_set_tiling(S.ctx, tiling)
    R = S.residual()
    torch.cuda.synchronize()
    sx, sy = S.flags()
    assert S.check() == 0
    S.close()
    Ro, sxo, syo, _ = O.residual(ocfg(P, recon=recon, order=order, riemann=riemann), P.Q,
                                 want_flags=True)
    e = res_err(R.cpu().numpy(), Ro, P).max()
    report(name, res_err=e)
    assert (sx == sxo).all() and (sy == syo).all()
    assert e <= (1e-6 if precision else 1e-12)


SCHEMES = {
    "prim": {}, "cons": {"recon": 1}, "order4": {"order": 4}, "cons4": {"recon": 1, "order": 4},
    "ss": {"riemann": 1}, "fp32": {"precision": gbr.GBR_PREC_FP32_BULK},
}


@pytest.mark.parametrize("scheme", sorted(SCHEMES))
@pytest.mark.parametrize("tiling,nx,ny", [
    (0, 656, 300), (0, 656, 310),      # 22 x 20 and 22 x 21 tiles of 31x15
    (1, 486, 461), (1, 486, 476),      # 33 x 31 and 33 x 32 tiles of 15x15
])
def test_forms_by_tile_count(tiling, nx, ny, scheme):
    kw = SCHEMES[scheme]
    check(f"{scheme} riemann{nx}x{ny} t{tiling}", PB.riemann(nx, seed=3, ny=ny), tiling, **kw)
    check(f"{scheme} noise{nx}x{ny} t{tiling}", noise(nx, ny, 0.0, PB.BC_PERIODIC), tiling, **kw)
    check(f"{scheme} noise visc{nx}x{ny} t{tiling}", noise(nx, ny, 1e-3, PB.BC_TRANSMISSIVE),
          tiling, **kw)


@pytest.mark.parametrize("precision", [gbr.GBR_PREC_FP64, gbr.GBR_PREC_FP32_BULK])
@pytest.mark.parametrize("tiling", range(4))
@pytest.mark.parametrize("nx,ny", [(12, 12), (13, 29), (31, 14), (46, 47), (127, 16)])
def test_small_and_ragged(nx, ny, tiling, precision):
    for mu in (0.0, 1e-3):
        for bc in (PB.BC_PERIODIC, PB.BC_TRANSMISSIVE):
            check(f"noise{nx}x{ny} mu={mu} bc={bc} t{tiling} p{precision}", noise(nx, ny, mu, bc),
                  tiling, precision=precision)
