"""Both sides of each line of the rule that serves the 15x15 shape by 15x7 tiles
or gives a lane one, two or four interfaces, on ragged grids, for every scheme that follows it.

Bars: as in the other residual tests (flags bit for bit, 1e-12 in FP64, 1e-6 in
FP32 bulk)."""
import pytest

from paper_2305_00762_amd import problems as PB
from test_line_forms_gpu import SCHEMES, check, noise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", sorted(SCHEMES))
@pytest.mark.parametrize("tx,ty", [(9, 11), (10, 10),       # 99, 100 tiles
                                   (20, 19), (20, 21),      # 380, 420
                                   (28, 28), (29, 28),      # 784, 812
                                   (43, 44), (44, 44)])     # 1892, 1936
def test_interfaces_per_lane(tx, ty, scheme):
    nx, ny = 15 * tx - 13, 15 * ty - 4                      # 2 and 11 cells in the last tiles
    kw = SCHEMES[scheme]
    check(f"{scheme} riemann{nx}x{ny}", PB.riemann(nx, seed=4, ny=ny), 1, **kw)
    check(f"{scheme} noise visc{nx}x{ny}", noise(nx, ny, 1e-3, PB.BC_PERIODIC), 1, **kw)
