"""A label outside [0, K) (GPU tier): log K and the gradient of the one-workgroup form and of the
one-column pass are those of the row tile, which an explicit tuning selects (a label outside the
16 padded classes has no term in log K)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n,p,K,pin", [(60, 5, 2, True), (60, 5, 4, True), (60, 5, 3, False), (40, 3, 9, True),
                                       (20000, 300, 2, True)])
def test_label_outside_the_classes(lib, n, p, K, pin, dtype):
    import torch
    rng = np.random.default_rng([n, p, K])
    X = torch.from_numpy(rng.normal(size=(n, p)).astype(dtype)).cuda()
    y = rng.integers(0, K, n).astype(np.int32)
    y[[1, 7, n - 1]] = -1, K, K + 100
    B = rng.normal(0.0, 0.3, size=(p, K)).astype(dtype)
    if pin:
        B[:, -1] = 0.0
    B, y = torch.from_numpy(B).cuda(), torch.from_numpy(y).cuda()
    logk, G = lib.logpost_grad(lib.Problem(X, y, K, pin_last_class=pin), B)
    want, Gw = lib.logpost_grad(lib.Problem(X, y, K, pin_last_class=pin, tuning=dict(path=1)), B)
    assert abs(float(logk) - float(want)) <= 1e-12 * abs(float(want))
    tol = 1e-12 if dtype == np.float64 else 1e-5
    assert float((G - Gw).double().norm()) <= tol * float(Gw.double().norm())
