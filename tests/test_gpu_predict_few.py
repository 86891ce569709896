"""Posterior-predictive classification with few samples (GPU tier), on both sides of the line between
the vector-unit form (first 0 to 10 samples at these sizes) and the matrix form: every class-block
count, pinned or not, rows and tiles with remainders, padded rows, non-finite rows. Tolerance as
in test_gpu_predict_layouts.py."""
import numpy as np
import pytest

import test_gpu_predict_layouts as layouts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [1, 2, 3, 5, 8, 11])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n,p,K,pin,pad", [
    (33, 70, 2, True, 0), (33, 70, 4, False, 1), (40, 130, 11, False, 0), (33, 20, 16, True, 2), (20, 64, 16, False, 0),
    (33, 70, 17, True, 0), (20, 33, 32, False, 3), (33, 130, 33, True, 0), (19, 50, 48, True, 0), (33, 40, 64, False, 0),
    (1500, 30, 10, True, 0), (5000, 8, 20, True, 1), (17, 1130, 2, True, 0), (1, 1, 3, False, 0)])
def test_few_samples(lib, n, p, K, pin, pad, S, dtype):
    layouts.test_layout_edges(lib, n, p, K, S, pin, pad, dtype)


@pytest.mark.parametrize("K,pin,S", [(10, True, 1), (10, False, 2), (20, True, 1), (64, False, 1)])
def test_nonfinite_rows_stay_in_their_rows(lib, K, pin, S):
    n, p = 32, 90
    X, samples = layouts._inputs(n, p, K, S, pin, 0, np.float32)
    mean0, cls0 = layouts._run(lib, X, p, samples, K, pin)
    X[3, 7], X[9, 89], X[20, 0] = np.inf, np.nan, -np.inf
    mean, cls = layouts._run(lib, X, p, samples, K, pin)
    bad = [3, 9, 20]
    good = np.setdiff1d(np.arange(n), bad)
    assert np.all(np.isnan(mean[bad])) and np.all(cls[bad] == 0)
    assert np.array_equal(mean[good], mean0[good]) and np.array_equal(cls[good], cls0[good])
