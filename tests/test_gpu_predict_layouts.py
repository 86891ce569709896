"""Posterior-predictive classification (GPU tier) at the edges of its two layouts: one class
block per free class up to 16 classes and 16-class blocks beyond, tiles of 16 rows, groups of 16
(or pairs of) samples, column groups with remainders, padded rows, both precisions; and rows
that hold an infinity or a NaN.

Tolerance. A logit is a sum of p products in the X precision, off by at most about
u p^(1/2) s with s^2 = sum_j (x_j b_j)^2 (u the unit roundoff; the errors of the partial sums,
each at most u/2 of a sum of size s, add like a random walk times p^(1/2)); the inputs have
s <= 2, and a probability moves by at most half of the largest logit error, plus 8 u for the
exponential and the sum. Over the worst of some thousand entries four times that:
4 u (p^(1/2) + 8)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SHAPES = [  # n, p, K, S, pinned, row padding
    (1, 1, 2, 1, True, 0), (16, 4, 2, 16, True, 0), (17, 65, 2, 33, False, 3), (15, 64, 3, 15, True, 1),
    (33, 63, 4, 65, True, 0), (40, 129, 5, 7, False, 0), (50, 785, 10, 100, True, 0), (31, 300, 11, 130, True, 5),
    (48, 17, 13, 66, False, 0), (18, 130, 15, 17, True, 0), (16, 16, 16, 16, True, 0), (35, 67, 16, 20, False, 2),
    (47, 70, 17, 3, True, 0), (16, 33, 32, 2, False, 0), (30, 130, 33, 1, True, 1), (19, 5, 48, 9, True, 0),
    (20, 60, 49, 4, False, 0), (33, 128, 64, 5, True, 0), (17, 1130, 2, 3, True, 0),
]


def _inputs(n, p, K, S, pin, pad, dtype):
    rng = np.random.default_rng([n, p, K, S])
    X = np.full((n, p + pad), np.nan, dtype=dtype)
    X[:, :p] = rng.normal(size=(n, p)).clip(-4, 4)
    samples = rng.normal(0.0, 0.4 / np.sqrt(p), size=(S, p, K)).astype(dtype)
    if pin:
        samples[:, :, -1] = 3.0                    # read as zero
    return X, samples


def _run(lib, X, p, samples, K, pin):
    import torch
    Xd = torch.from_numpy(X).cuda()[:, :p]
    mean, cls = lib.posterior_predictive(Xd, torch.from_numpy(samples).cuda(), K, pin)
    torch.cuda.synchronize()
    return mean.cpu().numpy(), cls.cpu().numpy()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n,p,K,S,pin,pad", SHAPES)
def test_layout_edges(lib, n, p, K, S, pin, pad, dtype):
    X, samples = _inputs(n, p, K, S, pin, pad, dtype)
    mean, cls = _run(lib, X, p, samples, K, pin)
    S64 = samples.astype(np.float64)
    if pin:
        S64[:, :, -1] = 0.0
    X64 = X[:, :p].astype(np.float64)
    want = np.mean([oracle.softmax_rows(oracle.logits(X64, B)) for B in S64], axis=0)
    tol = 4 * (2.0 ** -24 if dtype == np.float32 else 2.0 ** -53) * (np.sqrt(p) + 8)
    assert np.max(np.abs(mean - want)) <= tol
    top2 = np.sort(want, axis=1)[:, -2:]
    clear = top2[:, 1] - top2[:, 0] > 2 * tol
    assert np.array_equal(cls[clear], want.argmax(axis=1)[clear])


@pytest.mark.parametrize("K,pin", [(10, True), (10, False), (20, True)])
def test_nonfinite_rows_stay_in_their_rows(lib, K, pin):
    """A row with an infinity or a NaN has NaN probabilities and class 0; its tile's other rows
    are those of the finite data."""
    n, p, S = 32, 90, 18
    X, samples = _inputs(n, p, K, S, pin, 0, np.float32)
    mean0, cls0 = _run(lib, X, p, samples, K, pin)
    X[3, 7], X[9, 89], X[20, 0] = np.inf, np.nan, -np.inf
    mean, cls = _run(lib, X, p, samples, K, pin)
    bad = [3, 9, 20]
    good = np.setdiff1d(np.arange(n), bad)
    assert np.all(np.isnan(mean[bad])) and np.all(cls[bad] == 0)
    assert np.array_equal(mean[good], mean0[good]) and np.array_equal(cls[good], cls0[good])
