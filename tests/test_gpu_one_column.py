"""The pass for one free coefficient column (GPU tier): Poisson, probit and the pinned two-class
logit, at the edges of its 16-column blocks, load pieces and row pairs, with padded rows that hold
NaN. Bars: against the oracle, the element-wise bound of the row-sum rounding (16 u M) and rel-L2
1e-12 / 1e-5; against the row tile, whose float32 logits it forms in the same order, log K within
the rounding of a float64 sum of the n rows' terms (n u sum |l|, twice)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
# float64 problems are of the size from which the pass is taken
SHAPES = [(False, n, p, pad) for n, p, pad in [
    (1, 1024, 0), (2, 513, 0), (3, 1023, 1), (17, 512, 3), (33, 511, 0), (15, 1000, 8), (4099, 130, 2),
    (8200, 65, 0), (9000, 15, 1), (70000, 3, 0), (5001, 769, 7), (20011, 17, 0)]] + [
    (True, n, p, pad) for n, p, pad in [
        (2048, 512, 0), (2053, 511, 1), (4097, 257, 0), (10963, 192, 0), (10981, 191, 3), (32801, 65, 2), (131073, 16, 0),
        (700001, 3, 0)]]


@pytest.mark.parametrize("link", ["logit", "poisson", "probit"])
@pytest.mark.parametrize("f64,n,p,pad", SHAPES)
def test_edges(lib, f64, n, p, pad, link):
    import torch
    rng = np.random.default_rng([n, p])
    dtype = np.float64 if f64 else np.float32
    X = rng.normal(size=(n, p)).astype(dtype)
    B = rng.normal(0.0, 0.5 / np.sqrt(p), size=(p, 2 if link == "logit" else 1)).astype(dtype)
    if link == "logit":
        B[:, 1] = 0.0
    y = (rng.poisson(1.0, size=n) if link == "poisson" else rng.integers(0, 2, size=n)).astype(np.int32)
    buf = torch.full((n, p + pad), float("nan"), dtype=torch.float64 if f64 else torch.float32, device="cuda")
    buf[:, :p] = torch.from_numpy(X).cuda()
    code, code_o = dict(logit=(lib.HMC_LINK_SOFTMAX, oracle.SOFTMAX), poisson=(lib.HMC_LINK_POISSON, oracle.POISSON),
                        probit=(lib.HMC_LINK_PROBIT, oracle.PROBIT))[link]
    pin = link == "logit"
    args = (buf[:, :p], torch.from_numpy(y).cuda(), B.shape[1], 0, 1.0, pin)
    Bd = torch.from_numpy(B).cuda()
    logk, G = lib.logpost_grad(lib.Problem(*args, link=code), Bd)
    lk, g = float(logk), G.double().cpu().numpy()
    tile, _ = lib.logpost_grad(lib.Problem(*args, link=code, tuning=dict(path=1, waves=0, mb=0, grid=0, rows_per_slice=0)), Bd)
    X64, B64 = X.astype(np.float64), B.astype(np.float64)
    lk_o, G_o = oracle.log_kernel_and_grad(X64, y, B64, 0, 1.0, int(pin), code_o)
    assert np.linalg.norm(g - G_o) <= (1e-12 if f64 else 1e-5) * max(np.linalg.norm(G_o), 1.0)
    assert abs(lk - lk_o) <= (1e-12 if f64 else 1e-5) * max(abs(lk_o), 1.0)
    if pin:
        assert np.all(g[:, 1] == 0)
    if not f64:
        z = X64 @ B64[:, 0]
        terms = {"logit": np.logaddexp(0.0, np.abs(z)), "poisson": y * np.abs(z) + np.exp(z),
                 "probit": 1.0 + z * z}[link].sum() + 0.5 * (B64 ** 2).sum()
        assert abs(lk - float(tile)) <= 2 * (n + p) * 2.0 ** -53 * terms


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_row_that_is_not_finite(lib, bad):
    # the pinned class's logit sums x * 0: log K is NaN, as by the row tile, whatever the sign
    import torch
    rng = np.random.default_rng(3)
    X = rng.normal(size=(301, 600)).astype(np.float32)
    X[100, 77] = bad
    B = np.zeros((600, 2), np.float32)
    B[:, 0] = 0.1
    y = rng.integers(0, 2, size=301).astype(np.int32)
    args = (torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), 2)
    Bd = torch.from_numpy(B).cuda()
    logk, G = lib.logpost_grad(lib.Problem(*args), Bd)
    tile, Gt = lib.logpost_grad(lib.Problem(*args, tuning=dict(path=1, waves=0, mb=0, grid=0, rows_per_slice=0)), Bd)
    assert np.isnan(float(logk)) and np.isnan(float(tile))
    assert torch.equal(torch.isnan(G), torch.isnan(Gt))
