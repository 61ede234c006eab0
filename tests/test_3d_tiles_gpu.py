"""Every plane tile of the 3D stage (15x15, 16x16, 20x17, chosen by what their
tiles cost over the grid), exact and ragged, against the 3D oracle: flags bit
for bit, residuals to the bar of the other 3D residual tests."""
import pytest

from paper_2305_00762_amd import gbr
from paper_2305_00762_amd import problems as PB
from test_3d_gpu import check3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [7, 4])
@pytest.mark.parametrize("nx,ny,nz", [
    (15, 30, 400), (24, 35, 130),                 # 15x15 above one round of tiles
    (16, 16, 200), (32, 18, 140),                 # 16x16: exact, two rows over
    (20, 17, 200), (21, 34, 130), (39, 33, 90),   # 20x17: exact, a column over, ragged
])
def test_plane_tiles(nx, ny, nz, order):
    P = PB.riemann3d(nx, seed=nx, ny=ny, nz=nz)
    P.bc = (PB.BC_PERIODIC, PB.BC_TRANSMISSIVE, PB.BC_PERIODIC)
    assert check3(f"3d tiles {nx}x{ny}x{nz}", P, order=order, sweeps=gbr.GBR3_SWEEPS_LINES) > 0
