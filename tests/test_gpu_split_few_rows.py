"""Split-precision gradients of few rows (GPU tier), on both sides of the row counts up to which X goes
straight to the matrix operand: k steps with remainders, every class-block count, one and two planes,
NaN row padding. Against the FP64 oracle at the tolerance of the form."""
import numpy as np
import pytest

import oracle
from oracle import split

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hi_only", [False, True])
@pytest.mark.parametrize("n,p,K,pad", [
    (1, 1, 2, 7), (1, 40, 20, 8), (3, 31, 5, 1), (15, 32, 16, 0), (16, 33, 17, 7), (33, 96, 33, 8), (64, 128, 8, 0),
    (65, 129, 32, 7), (80, 1000, 10, 24), (81, 1000, 10, 24), (80, 257, 64, 7), (127, 513, 40, 7), (128, 300, 64, 4),
    (129, 300, 64, 4), (7, 5003, 3, 5)])
def test_gradient(lib, n, p, K, pad, hi_only):
    import torch
    rng = np.random.default_rng([n, p, K])
    X = rng.normal(size=(n, p)).astype(np.float32)
    y = rng.integers(0, K, n).astype(np.int32)
    B = rng.normal(0.0, 0.5 / np.sqrt(p), size=(p, K)).astype(np.float32)
    B[:, -1] = 0.0
    h, l = lib.split_bf16(torch.from_numpy(X).cuda(), hi_only=hi_only)
    planes = []
    for plane in (h, l):
        buf = torch.full((n, p + pad), float("nan"), dtype=torch.bfloat16, device="cuda")
        if plane is not None:
            buf[:, :p] = plane
        planes.append(buf[:, :p])
    assert (p + pad) % 8 == 0
    prob = lib.Problem(planes[0], torch.from_numpy(y).cuda(), K, X_lo=None if hi_only else planes[1])
    logk, G = lib.logpost_grad(prob, torch.from_numpy(B).cuda())
    xh, xl = split.split_hilo(X)
    Xe, B64 = xh if hi_only else xh + xl, B.astype(np.float64)
    lk, Go = oracle.log_kernel_and_grad(Xe, y, B64, 0, 1.0, 1)
    g = G.double().cpu().numpy()
    assert np.linalg.norm(g - Go) <= 6e-5 * max(np.linalg.norm(Go), 1e-3)
    assert abs(float(logk) - lk) <= 2.0 ** -14 * float(np.sum(np.max(np.abs(Xe) @ np.abs(B64), axis=1))) + n * 1e-6
    assert np.all(g[:, -1] == 0)


@pytest.mark.parametrize("chains,hi_only", [(1, False), (2, False), (4, False), (1, True), (4, True)])
@pytest.mark.parametrize("shapes", [[(1, 40, 2), (33, 97, 16), (80, 300, 5)], [(7, 1030, 9), (81, 64, 3)], [(128, 65, 4), (2, 33, 7)]])
def test_batch(lib, shapes, chains, hi_only):
    import torch
    rng = np.random.default_rng(len(shapes) + chains)
    probs, mats, ys = [], [], []
    for n, p, K in shapes:
        X = rng.normal(size=(n, p)).astype(np.float32)
        y = rng.integers(0, K, n).astype(np.int32)
        h, l = lib.split_bf16(torch.from_numpy(X).cuda(), hi_only=hi_only)
        probs.append(lib.Problem(h, torch.from_numpy(y).cuda(), K, X_lo=l))
        xh, xl = split.split_hilo(X)
        mats.append(xh if hi_only else xh + xl)
        ys.append(y)
    bt = lib.Batch(probs, chains)
    B, G, logk = bt.zeros_state()
    for b in B:
        b.copy_(torch.from_numpy(rng.normal(0.0, 0.3, size=tuple(b.shape)).astype(np.float32) / np.sqrt(b.shape[1])))
        b[..., -1] = 0.0
    bt.logpost_grad(B, G, logk)
    for b, (Xe, y) in enumerate(zip(mats, ys)):
        for c in range(chains):
            B64 = B[b][c].double().cpu().numpy()
            lk, Go = oracle.log_kernel_and_grad(Xe, y, B64, 0, 1.0, 1)
            assert np.linalg.norm(G[b][c].double().cpu().numpy() - Go) <= 6e-5 * max(np.linalg.norm(Go), 1e-3)
            assert abs(float(logk[b, c]) - lk) <= 2.0 ** -14 * float(np.sum(np.max(np.abs(Xe) @ np.abs(B64), axis=1))) + 1e-4
