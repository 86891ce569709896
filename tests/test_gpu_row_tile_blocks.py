"""Row tile (GPU tier) where the last 16-column blocks of some or all waves lie past column p: one
block below, at and above each count of blocks per wave that has a loop of its own (a half, three
quarters and all of the variant's), for every class-block count and both precisions, with the path
forced. Bars: the element-wise bound of the row-sum rounding (16 u M) and rel-L2 1e-12 / 1e-5."""
import numpy as np
import pytest

import oracle
from gradbound import UNIT_ROUNDOFF, assert_elementwise

pytestmark = pytest.mark.gpu

CASES = ([("f32", p, 10, pad) for p, pad in [
    (257, 0), (258, 2), (496, 0), (511, 1), (512, 0), (513, 0), (528, 0), (529, 3), (753, 0), (768, 0), (769, 0),
    (785, 0), (800, 8), (1009, 0), (1024, 0)]]
    + [("f32", p, 20, pad) for p, pad in [(129, 0), (250, 1), (257, 0), (369, 0), (384, 0), (385, 2), (512, 0)]]
    + [("f32", p, 40, pad) for p, pad in [(129, 0), (256, 0), (257, 0), (384, 4), (385, 0)]]
    + [("f64", p, 3, pad) for p, pad in [(129, 0), (240, 1), (257, 0), (384, 0), (385, 0), (400, 2), (511, 0), (512, 0)]]
    + [("f64", p, 20, pad) for p, pad in [(113, 0), (129, 1), (250, 0)]])


@pytest.mark.parametrize("xfmt,p,K,pad", CASES)
def test_blocks_past_p(lib, xfmt, p, K, pad):
    import torch
    n = 333
    rng = np.random.default_rng([p, K])
    dtype = np.float64 if xfmt == "f64" else np.float32
    X = rng.normal(size=(n, p)).astype(dtype)
    y = rng.integers(0, K, size=n).astype(np.int32)
    B = rng.normal(0.0, 0.5 / np.sqrt(p), size=(p, K)).astype(dtype)
    B[:, -1] = 0.0
    buf = torch.full((n, p + pad), float("nan"), dtype=torch.float64 if xfmt == "f64" else torch.float32, device="cuda")
    buf[:, :p] = torch.from_numpy(X).cuda()
    # five workgroups: a chain of tiles in each
    prob = lib.Problem(buf[:, :p], torch.from_numpy(y).cuda(), K, tuning=dict(path=1, waves=0, mb=0, grid=5, rows_per_slice=0))
    logk, G = lib.logpost_grad(prob, torch.from_numpy(B).cuda())
    X64, B64 = X.astype(np.float64), B.astype(np.float64)
    lk, Go = oracle.log_kernel_and_grad(X64, y, B64)
    g = G.double().cpu().numpy()
    tol = 1e-12 if xfmt == "f64" else 1e-5
    assert np.linalg.norm(g - Go) <= tol * np.linalg.norm(Go)
    assert_elementwise(g, Go, X64, y, B64, 0, 1.0, 1, UNIT_ROUNDOFF[xfmt])
    assert abs(float(logk) - lk) <= tol * abs(lk)
