"""Split-precision encoding over the sizes at which its work split changes (GPU tier): one group of 8
columns per thread or more, rows in one piece or several, fewer than 8 columns, padded sources and
planes, infinities and NaN. Both planes equal the oracle's bit for bit (rows repeat a block that the
oracle encodes), padding columns are zero."""
import numpy as np
import pytest

from oracle import split

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n,p,pad,extra", [
    (1, 1, 0, 0), (3, 2047, 1, 8), (2, 8474, 0, 0), (1, 70001, 0, 0), (33, 7, 5, 0), (70001, 1, 0, 56), (40000, 3, 1, 8),
    (257, 255, 0, 0), (300, 257, 3, 64), (9000, 470, 0, 0), (8193, 1031, 1, 0), (2100, 4100, 0, 24), (17000, 2049, 0, 0)])
def test_planes(lib, n, p, pad, extra, dtype):
    import torch
    rng = np.random.default_rng([n, p])
    m = min(n, 61)
    X = rng.standard_normal((m, p)) * np.exp2(rng.integers(-140, 120, (m, p)))
    special = [np.inf, -np.inf, np.nan, 0.0, -0.0, 3.4e38, 1e-45]
    at = rng.choice(X.size, min(len(special), X.size), replace=False)
    X.flat[at] = special[:len(at)]
    X = X.astype(dtype)
    with np.errstate(invalid="ignore", over="ignore"):
        want = split.split_hilo(X.astype(np.float64))
    rows = torch.arange(n, device="cuda") % m
    buf = torch.full((n, p + pad), 7.0, dtype=torch.from_numpy(X).dtype, device="cuda")
    buf[:, :p] = torch.from_numpy(X).cuda()[rows]
    ldo = (p + 7) // 8 * 8 + extra
    hi = torch.full((n, ldo), 5.0, dtype=torch.bfloat16, device="cuda")
    lo = torch.full((n, ldo), 5.0, dtype=torch.bfloat16, device="cuda")
    code = lib.HMC_X_F64 if dtype == np.float64 else lib.HMC_X_F32
    lib.hmc_split_bf16(buf, code, n, p, p + pad, hi, lo, ldo)
    for got, w in zip((hi, lo), want):
        assert np.array_equal(got[:m, :p].double().cpu().numpy(), w, equal_nan=True)
        assert not bool(got[:, p:].float().any())
        bits = got.view(torch.int16)
        assert torch.equal(bits, bits[rows])
    only = torch.full((n, ldo), 5.0, dtype=torch.bfloat16, device="cuda")
    lib.hmc_split_bf16(buf, code, n, p, p + pad, only, None, ldo)
    assert torch.equal(only.view(torch.int16), hi.view(torch.int16))
