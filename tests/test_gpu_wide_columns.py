"""Wide-p gradient (GPU tier) at the edges of its column spans (16 columns per wave, or 256 bytes of
a row where the workgroups are many; four waves per workgroup), row tiles and slices: remainders of both, odd tile counts per slice, padded
rows with NaN, every class-block count, both precisions, with the path forced. Bars: the
element-wise bound of the row-sum rounding (16 u M) and rel-L2 1e-12 / 1e-5."""
import numpy as np
import pytest

import oracle
from gradbound import UNIT_ROUNDOFF, assert_elementwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("n,p,K,pad,rows", [
    (1, 1, 2, 0, 0), (15, 31, 3, 1, 0), (16, 32, 16, 0, 0), (17, 33, 17, 3, 0), (33, 63, 5, 0, 64), (64, 64, 33, 0, 64),
    (65, 65, 64, 5, 64), (100, 127, 4, 0, 0), (130, 129, 20, 0, 64), (200, 255, 7, 1, 128), (333, 257, 40, 0, 128),
    (79, 1025, 10, 2, 64), (48, 1023, 2, 0, 0), (500, 513, 16, 0, 192), (96, 2050, 12, 6, 0),
    # workgroups enough for the wider spans (64 and 32 columns per wave)
    (1300, 5103, 5, 0, 64), (1999, 4961, 20, 1, 64), (2001, 5000, 40, 0, 64),
])
def test_span_edges(lib, n, p, K, pad, rows, f64):
    import torch
    rng = np.random.default_rng([n, p, K])
    dtype = np.float64 if f64 else np.float32
    X = rng.normal(size=(n, p)).astype(dtype)
    y = rng.integers(0, K, size=n).astype(np.int32)
    B = rng.normal(0.0, 0.5 / np.sqrt(p), size=(p, K)).astype(dtype)
    B[:, -1] = 0.0
    buf = torch.full((n, p + pad), float("nan"), dtype=torch.float64 if f64 else torch.float32, device="cuda")
    buf[:, :p] = torch.from_numpy(X).cuda()
    prob = lib.Problem(buf[:, :p], torch.from_numpy(y).cuda(), K,
                       tuning=dict(path=2, waves=0, mb=0, grid=0, rows_per_slice=rows))
    logk, G = lib.logpost_grad(prob, torch.from_numpy(B).cuda())
    X64, B64 = X.astype(np.float64), B.astype(np.float64)
    lk, Go = oracle.log_kernel_and_grad(X64, y, B64)
    g = G.double().cpu().numpy()
    assert np.linalg.norm(g - Go) <= (1e-12 if f64 else 1e-5) * np.linalg.norm(Go)
    assert_elementwise(g, Go, X64, y, B64, 0, 1.0, 1, UNIT_ROUNDOFF["f64" if f64 else "f32"])
    assert abs(float(logk) - lk) <= (1e-12 if f64 else 1e-5) * abs(lk)
