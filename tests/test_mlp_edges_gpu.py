"""Feature blocks and minibatch forms of the learned detector at their edges:
grids that end inside a 32 x 8 block or are smaller than its halo, both boundary
types; batches on both sides of the one-group-per-wave form, that end inside a
group, and the largest.  Bars: features and labels bit for bit, gradients within
1e-4 per block, norm-wise (the bf16 operands' bar of the other gradient tests)."""
import numpy as np
import pytest

import oracle as O
import oracle.mlp as M
from paper_2305_00762_amd import gbr
from paper_2305_00762_amd import problems as PB
from gpu_util import ocfg, report, require_gpu
from test_mlp_gpu import gpu_features, make_net

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", [PB.BC_PERIODIC, PB.BC_TRANSMISSIVE])
@pytest.mark.parametrize("nx,ny", [(12, 12), (32, 16), (33, 17), (63, 13), (95, 40)])
def test_feature_blocks(nx, ny, bc):
    P = PB.riemann(nx, seed=nx, ny=ny, split=(0.45, 0.55))
    P.bc_x = P.bc_y = bc
    f, chi = gpu_features(P)
    fo = np.concatenate([M.features(P.Q, bc, bc, P.gamma, direction=d) for d in (0, 1)])
    _, px, py = O.cell_flags(ocfg(P), P.Q)
    assert (f == fo).all()
    assert (chi == np.concatenate([c.ravel() for c in M.labels(px, py)])).all()


@pytest.mark.parametrize("batch", [1, 65, 16384, 16385, 65536])
def test_gradient_forms(batch):
    torch = require_gpu()
    P = PB.riemann(96, seed=3)
    f, chi = gpu_features(P)
    m, w, b = make_net(2)
    idx = PB.balanced_batches(chi, batch, 1, seed=9)[0]
    g = torch.empty(2018, dtype=torch.float32, device="cuda")
    gbr.gbr_mlp_grad(m, torch.from_numpy(f.view(np.int16)).cuda(), torch.from_numpy(chi).cuda(),
                     torch.from_numpy(idx).cuda(), batch, g)
    torch.cuda.synchronize()
    gbr.gbr_mlp_destroy(m)
    g = g.cpu().numpy().astype(np.float64)
    loss, dw, db = M.loss_and_grad(f[idx], chi[idx], w, b, round_ops=True)
    ref = np.concatenate([dw, db])
    for a, e in ((0, 896), (896, 1920), (1920, 1952), (1952, 2017)):
        n = np.linalg.norm(ref[a:e])
        rel = np.linalg.norm(g[a:e] - ref[a:e]) / (n if n > 0 else 1.0)
        report(f"grad [{a}:{e}] B={batch}", rel=rel)
        assert rel <= 1e-4
    assert abs(g[2017] / batch - loss) <= 1e-4 * abs(loss)
