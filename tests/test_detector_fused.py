"""The line kernels take the detector's decision psi < 1/2 as one fused
operation, fl(4 ab + 2 eps) < den on fl(ab) (Sec. 2.4, eq. buffer).  It equals
the decision of the division in IEEE double arithmetic: 4 ab is exact, so numpy
rounds 4 ab + 2 eps once as the device's fused operation does."""
import numpy as np
import pytest

import oracle as O


@pytest.mark.parametrize("scale", [1e-160, 1e-9, 1e-6, 1e-3, 1.0, 1e3, 1e150])
def test_fused_decision_is_the_division(scale):
    eps = O.detector_eps()
    rng = np.random.default_rng(7)
    b = scale * 10.0 ** rng.uniform(-1, 1, (2000, 1))
    t = 2.0 * b - np.sqrt(3.0 * b * b + eps)          # psi = 1/2 at a = t
    a = np.concatenate([np.abs(t) + np.arange(-50, 51) * np.spacing(np.abs(t)),
                        b * 10.0 ** rng.uniform(-3, 3, (2000, 100))], axis=1)
    a, b = np.abs(a), np.broadcast_to(b, a.shape)
    num = 2.0 * (a * b) + eps
    den = (a * a + b * b) + eps
    want = num / den < 0.5
    got = 4.0 * (a * b) + 2.0 * eps < den
    assert (got == want).all()
    if 1e-3 <= scale:
        assert want.any() and not want.all()
