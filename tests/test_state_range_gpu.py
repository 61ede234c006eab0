"""States of any magnitude: density and pressure far from one, on their own and
together, through every Riemann solver.

The Euler equations scale: rho and p by s leave the velocities and multiply
every flux by s; p by s alone multiplies the velocities by sqrt(s).  So the bars
are those of the unscaled fields: flags bit for bit and a residual within 1e-12
(FP64) or 1e-6 (FP32 bulk) of the flux-divergence scale.  FP32 bulk: the scales
at which the fluxes themselves, rho c^3 among them, are normal float32 numbers."""
import pytest

from paper_2305_00762_amd import gbr
from paper_2305_00762_amd import problems as PB
from test_line_forms_gpu import check, noise

pytestmark = pytest.mark.gpu


def scaled(kind, nx, ny, rho, p):
    """A vortex (smooth) or noise (nearly all interfaces flagged), its density
    and pressure multiplied."""
    P = PB.vortex(nx, ny=ny) if kind == "vortex" else noise(nx, ny, 0.0, PB.BC_PERIODIC)
    r, u, v = P.Q[0], P.Q[1] / P.Q[0], P.Q[2] / P.Q[0]
    pr = (P.gamma - 1) * (P.Q[3] - 0.5 * r * (u * u + v * v))
    s = (p / rho) ** 0.5
    P.Q = PB.prim_to_state(r * rho, u * s, v * s, pr * p, P.gamma)
    return P


@pytest.mark.parametrize("kind", ["vortex", "noise"])
@pytest.mark.parametrize("rho,p", [(1e-25, 1e-25), (1e25, 1e25), (1e-30, 1e-30), (1e30, 1e30),
                                   (1e-20, 1e-24), (1e20, 1e24), (1e-25, 1e-16), (1e25, 1e16)])
def test_fp32_bulk(kind, rho, p):
    P = scaled(kind, 50, 37, rho, p)
    for tiling in (0, 1):
        check(f"fp32 {kind} rho {rho:g} p {p:g} t{tiling}", P, tiling,
              precision=gbr.GBR_PREC_FP32_BULK)
