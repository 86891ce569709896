"""Split-precision passes on planes beyond 4 GiB whose rows are padded with NaN (GPU tier).

p is a multiple of 8 but not of 32, so the last k step of the logits holds whole 16-byte pieces
past column p, and with the row pitch a power of two the last bytes that a 32-bit offset reaches
are row padding too. No padding element may reach log K or the gradient: against the FP64 oracle
at the tolerance of the form."""
import numpy as np
import pytest

import oracle
from oracle import split
from workloads import make_problem, make_random_state

pytestmark = pytest.mark.gpu

LDX = 1 << 22


def _planes(lib, prob, n, p, hi_only):
    """(hi, lo) of X in rows of LDX elements, NaN past column p, and the matrix they hold."""
    import torch
    hi = torch.full((n, LDX), float("nan"), dtype=torch.bfloat16, device="cuda")
    lo = None if hi_only else torch.full((n, LDX), float("nan"), dtype=torch.bfloat16, device="cuda")
    h, l = lib.split_bf16(torch.from_numpy(np.ascontiguousarray(prob.X64)).cuda(), hi_only=hi_only)
    hi[:, :p] = h
    if lo is not None:
        lo[:, :p] = l
    assert hi.numel() * 2 > 1 << 32
    xh, xl = split.split_hilo(prob.X64)
    return hi[:, :p], None if lo is None else lo[:, :p], xh if hi_only else xh + xl


def _check(prob, X, B, logk, G):
    Bs = B.double().cpu().numpy()
    Gd = G.double().cpu().numpy()
    lk, Go = oracle.log_kernel_and_grad(X, prob.y, Bs, prob.prior, prob.prior_scale, 1)
    assert np.all(np.isfinite(Gd)) and np.isfinite(logk)
    assert np.linalg.norm(Gd - Go) <= 6e-5 * np.linalg.norm(Go)
    assert abs(logk - lk) <= 2.0 ** -14 * float(np.sum(np.max(np.abs(X) @ np.abs(Bs), axis=1))) + len(X) * 1e-6


@pytest.mark.parametrize("n,p,K,hi_only", [(700, 1000, 5, True), (700, 1000, 40, False), (600, 8, 20, True)])
def test_single(lib, n, p, K, hi_only):
    import torch
    prob = make_problem("c4_bf16", n=n, p=p, K=K)
    hi, lo, X = _planes(lib, prob, n, p, hi_only)
    dp = lib.Problem(hi, torch.from_numpy(prob.y).cuda(), K, prob.prior, prob.prior_scale, True, X_lo=lo)
    B = torch.from_numpy(make_random_state(prob, 0.05).astype(np.float32)).cuda()
    logk, G = lib.logpost_grad(dp, B)
    _check(prob, X, B, float(logk), G)
    del dp, hi, lo
    torch.cuda.empty_cache()


def test_batched(lib):
    import torch
    probs, dev, mats = [], [], []
    for n, p, K in ((700, 1000, 5), (650, 24, 9)):
        prob = make_problem("c4_bf16", n=n, p=p, K=K)
        hi, lo, X = _planes(lib, prob, n, p, False)
        probs.append(prob)
        mats.append(X)
        dev.append(lib.Problem(hi, torch.from_numpy(prob.y).cuda(), K, prob.prior, prob.prior_scale, True, X_lo=lo))
    bt = lib.Batch(dev, 4)
    B, G, logk = bt.zeros_state()
    for b, prob in enumerate(probs):
        for c in range(4):
            B[b][c].copy_(torch.from_numpy(make_random_state(prob, 0.1, seed=10 * b + c).astype(np.float32)))
    bt.logpost_grad(B, G, logk)
    for b, prob in enumerate(probs):
        for c in range(4):
            _check(prob, mats[b], B[b][c], float(logk[b, c]), G[b][c])
    del bt, dev, hi, lo
    torch.cuda.empty_cache()
