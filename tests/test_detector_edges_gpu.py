"""The kernels' detector decision where psi is within a few ulp of 1/2: density
rows built from pairs of one-sided variations (a, b) on both sides of the
threshold, the flags compared bit for bit with the oracle's division -- exported
by the stage kernels (2D, 3D) and as the plain labels of gbr_mlp_features."""
import numpy as np
import pytest

import oracle as O
from paper_2305_00762_amd import gbr
from paper_2305_00762_amd import problems as PB
from gpu_util import gpu_residual, ocfg, require_gpu

pytestmark = pytest.mark.gpu

N, ROWS = 30, 481


def density(scale, offset):
    """Rows of five jumps b and five jumps -a in turn.  Beside a change of slope one
    variation is b (or a) with a second difference of a + b on the other side, so
    psi passes 1/2 near a = 2 b - sqrt(3 b^2 + eps) and its mirror image; every
    other row moves a by a few ulp of the densities."""
    rng = np.random.default_rng(3)
    eps = O.detector_eps()
    r = np.empty((ROWS, N))
    for i in range(ROWS):
        b = scale * 2.0 ** rng.uniform(-2, 2)
        a = abs(2.0 * b - np.sqrt(3.0 * b * b + eps))
        k = i % 9 - 4
        a += k * np.spacing(max(a, offset)) if i % 2 else 0.0
        d = np.zeros(N - 1)
        for c in range(0, N - 1, 10):
            d[c:c + 5], d[c + 5:c + 10] = b, -abs(a)
        r[i] = offset + np.concatenate([[0.0], np.cumsum(d)])
    return r


def psi(r):
    """The detector's psi along rows, cells 2 .. N - 3 (Sec. 2.4)."""
    a = np.abs(r[:, 2:-2] - r[:, 1:-3]) + np.abs(r[:, 2:-2] - 2 * r[:, 1:-3] + r[:, :-4])
    b = np.abs(r[:, 2:-2] - r[:, 3:-1]) + np.abs(r[:, 2:-2] - 2 * r[:, 3:-1] + r[:, 4:])
    e = O.detector_eps()
    return (2 * a * b + e) / (a * a + b * b + e)


@pytest.mark.parametrize("scale,offset", [(0.3, 1.0), (0.05, 1.0), (1e-3, 1.0), (300.0, 1024.0)])
def test_flags_at_the_threshold(scale, offset):
    from paper_2305_00762_amd.solver import Solver
    torch = require_gpu()
    r = density(scale, offset)
    assert (r > 0).all()
    assert (np.abs(psi(r) - 0.5) < 1e-9).any()
    for T in (False, True):                         # along x, along y
        rho = np.ascontiguousarray(r.T if T else r)
        ny, nx = rho.shape
        P = PB.free_stream(nx, ny=ny, bc=PB.BC_TRANSMISSIVE)
        P.Q = PB.prim_to_state(rho, 0 * rho, 0 * rho, 0 * rho + 1.0)
        _, ox, oy, _ = O.residual(ocfg(P), P.Q, want_flags=True)
        assert 0 < (ox if not T else oy).mean() < 1
        for kw in ({}, {"precision": gbr.GBR_PREC_FP32_BULK}, {"recon": 1}, {"mp_mode": 1}):
            _, sx, sy, st = gpu_residual(P, **kw)
            assert st == gbr.GBR_OK
            assert (sx == ox).all() and (sy == oy).all(), kw
        _, px, py = O.cell_flags(ocfg(P), P.Q)
        S = Solver(P)
        feat = torch.zeros((2 * nx * ny, 32), dtype=torch.int16, device="cuda")
        chi = torch.zeros(2 * nx * ny, dtype=torch.uint8, device="cuda")
        gbr.gbr_mlp_features(S.ctx, S.Q, feat, chi)
        torch.cuda.synchronize()
        got = chi.cpu().numpy().reshape(2, ny, nx)
        assert (got[0] == (px < 0.5)).all() and (got[1] == (py < 0.5)).all()
        S.close()


def test_flags_at_the_threshold_3d():
    from paper_2305_00762_amd.solver import Solver3
    torch = require_gpu()
    rows = density(0.3, 1.0)[:240]
    for axis in range(3):                           # the rows along x, y, z
        rho = np.broadcast_to(rows, (12,) + rows.shape)
        rho = np.ascontiguousarray(np.moveaxis(rho, 2, 2 - axis))
        nz, ny, nx = rho.shape
        P = PB.riemann3d(nx, ny=ny, nz=nz)
        z = 0 * rho
        P.Q = PB.prim_to_state3(rho, z, z, z, z + 1.0)
        want = O.residual3(O.make_cfg3(nx, ny, nz, *P.geometry(), bc=P.bc, gamma=P.gamma), P.Q,
                           want_flags=True)[1:]
        S = Solver3(P, export_flags=True)
        S.residual()
        torch.cuda.synchronize()
        assert 0 < want[axis].mean() < 1
        assert all((a == b).all() for a, b in zip(S.flags(), want))
        S.close()
