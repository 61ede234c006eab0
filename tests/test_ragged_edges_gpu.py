"""Lanes are dealt over the cells of a tile that are inside the grid: every
remainder a ragged edge can have, in every tile shape, on a field that flags
almost every interface.

Bars: detector flags bit for bit; residuals within 1e-12 of the flux-divergence
scale max|F|/dx, the bar the other residual tests derive."""
import pytest

from test_line_forms_gpu import check, noise, require_gpu
from paper_2305_00762_amd import gbr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiling", range(4))
@pytest.mark.parametrize("mu", [0.0, 1e-3])
def test_every_remainder(tiling, mu):
    require_gpu()
    from paper_2305_00762_amd.solver import Solver
    S = Solver(noise(64, 64, mu, 0))
    gbr.gbr_set_tiling(S.ctx, tiling)
    _, tx, ty = gbr.gbr_get_tiling(S.ctx)
    S.close()
    for k in range(max(tx, ty)):
        nx, ny = tx + 1 + k % tx, 2 * ty + 1 + (k * 7) % ty
        check(f"ragged t{tiling} {nx}x{ny}", noise(max(nx, 12), ny, mu, k % 2), tiling)


@pytest.mark.parametrize("rx,ry", [(1, 14), (4, 1), (3, 8), (15, 2), (30, 5)])
def test_four_interfaces_a_lane(rx, ry):
    """Grids of enough tiles for the four-interface form."""
    check(f"ragged K=4 31x15 {rx} {ry}", noise(31 * 21 + rx, 15 * 22 + ry, 0.0, 1), 0)
    check(f"ragged K=4 15x15 {rx} {ry}", noise(15 * 33 + rx % 15, 15 * 33 + ry, 0.0, 0), 1)
