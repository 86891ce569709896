"""Split-precision encoding (GPU tier) at the edges of its kernel: column groups with
remainders, rows of one group and rows longer than a workgroup's share, padded rows, the hi
plane alone; and values around the bfloat16 range, ties, infinities and NaN. The planes must
equal the oracle's encodings bit for bit (a NaN keeps its sign and becomes quiet)."""
import warnings

import numpy as np
import pytest

from oracle import split

pytestmark = pytest.mark.gpu


def _values(rng, n, p, dtype):
    """Random values of every exponent around the range, with short and long significands."""
    e = rng.integers(-150, 131, size=(n, p))
    m = 1.0 + rng.integers(0, 2 ** 52, size=(n, p)) * 2.0 ** -52
    short = rng.random((n, p))
    m = np.where(short < 0.3, np.round(m * 256) / 256, m)          # ties of eight bits
    m = np.where((short > 0.3) & (short < 0.4), np.round(m * 128) / 128 + 2.0 ** -40, m)
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")
        x = (np.ldexp(m, e) * rng.choice([-1.0, 1.0], size=(n, p))).astype(dtype)
        special = np.array([0.0, -0.0, np.inf, -np.inf, 1e-45, -3.4028235e38, 3.39e38, 2.0 ** -134, 1.5 * 2.0 ** -133,
                            5e-324, 1e300], dtype=np.float64).astype(dtype)
    x.reshape(-1)[:special.size] = special[:x.size]
    return x


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n,p,pad,ldo,lo", [
    (1, 1, 0, 8, True), (5000, 7, 0, 8, True), (257, 9, 3, 16, False), (3, 2049, 0, 2056, True),
    (2, 20000, 1, 20032, True), (301, 64, 0, 64, True), (33, 1000, 24, 1024, True), (700, 127, 1, 128, False),
])
def test_split_edges(lib, n, p, pad, ldo, lo, dtype):
    import torch
    x = _values(np.random.default_rng([n, p]), n, p, dtype)
    buf = torch.full((n, p + pad), float("nan"), dtype=torch.from_numpy(x).dtype, device="cuda")
    buf[:, :p] = torch.from_numpy(x).cuda()
    hi = torch.full((n, ldo), -1, dtype=torch.int16, device="cuda")
    lw = torch.full((n, ldo), -1, dtype=torch.int16, device="cuda")
    lib.hmc_split_bf16(buf, lib.HMC_X_F64 if dtype == np.float64 else lib.HMC_X_F32, n, p, p + pad, hi,
                       lw if lo else None, ldo)
    torch.cuda.synchronize()
    hb, lb = hi.cpu().numpy().view(np.uint16), lw.cpu().numpy().view(np.uint16)
    with np.errstate(invalid="ignore"):
        ho, lo_ = split.split_hilo(x.astype(np.float64))
    assert np.array_equal(hb[:, :p], split.bf16_bits(ho)) and not hb[:, p:].any()
    if lo:
        fine = ~np.isnan(lo_)
        assert np.array_equal(lb[:, :p][fine], split.bf16_bits(lo_)[fine]) and not lb[:, p:].any()
        assert np.all(lb[:, :p][~fine] & 0x7FFF == 0x7FC0)         # inf - inf
    else:
        assert np.all(lb == 0xFFFF)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_split_nan(lib, dtype):
    import torch
    x = torch.tensor([[np.nan, -np.nan, 1.0]], dtype=torch.float64).to(torch.float64 if dtype == np.float64 else torch.float32)
    hi, _ = lib.split_bf16(x.cuda())
    assert hi.cpu().contiguous().view(torch.int16).numpy().view(np.uint16).tolist() == [[0x7FC0, 0xFFC0, 0x3F80]]
