"""Split-precision passes (GPU tier) at the edges of their tiles: 64-column chunks of X, 32-column
k steps and 128-column blocks with remainders, 16-, 32- and 128-row blocks with remainders, one, two
and four class blocks, rows on and off 128-byte lines (NaN in the padding), and an X larger than
the part kept in the memory-side cache. Bars as for the form's other shapes: gradient rel-L2
6e-5 (about 4 * 2^-16) against the oracle on the values the planes hold, log K within
2^-14 sum_i max_k sum_j |x_ij b_jk| + n * 1e-6."""
import numpy as np
import pytest

import oracle
from oracle import split

pytestmark = pytest.mark.gpu
GTOL = 6e-5


def _check(lib, n, p, K, hi_only, ldx, reps=1):
    import torch
    rng = np.random.default_rng([n, p, K])
    X = rng.normal(size=(n, p)).astype(np.float32)
    y = rng.integers(0, K, size=n).astype(np.int32)
    B = rng.normal(0.0, 0.5 / np.sqrt(p), size=(p, K)).astype(np.float32)
    planes = []
    for plane in split.split_hilo(X.astype(np.float64))[:1 if hi_only else 2]:
        t = torch.full((n, ldx), float("nan"), dtype=torch.bfloat16, device="cuda")
        t[:, :p] = torch.from_numpy(plane.astype(np.float32)).cuda().to(torch.bfloat16)
        planes.append(t[:, :p])
    prob = lib.Problem(planes[0], torch.from_numpy(y).cuda(), K, X_lo=None if hi_only else planes[1])
    logk, G = lib.logpost_grad(prob, torch.from_numpy(B).cuda())
    first = G.clone()
    for _ in range(reps):
        logk, G = lib.logpost_grad(prob, torch.from_numpy(B).cuda())
    assert torch.equal(first, G)
    hi, lo = split.split_hilo(X.astype(np.float64))
    Xe = hi if hi_only else hi + lo
    B64 = B.astype(np.float64)
    B64[:, -1] = 0.0
    lk, Go = oracle.log_kernel_and_grad(Xe, y, B64)
    err = np.linalg.norm(G.double().cpu().numpy() - Go) / np.linalg.norm(Go)
    bound = n * 1e-6 + \
        2.0 ** -14 * float(np.sum(np.max(np.abs(Xe) @ np.abs(B64), axis=1)))
    assert err <= GTOL and abs(float(logk) - lk) <= bound, (err, float(logk) - lk, bound)


@pytest.mark.parametrize("hi_only", [False, True])
@pytest.mark.parametrize("n,p,K", [
    (1, 1, 2), (15, 31, 3), (16, 32, 16), (17, 33, 17), (31, 63, 32), (32, 64, 33), (33, 65, 64), (127, 127, 5),
    (128, 128, 16), (129, 129, 20), (257, 191, 64), (1000, 193, 9), (2049, 256, 40), (300, 257, 2), (161, 1000, 48),
])
def test_tile_edges(lib, n, p, K, hi_only):
    _check(lib, n, p, K, hi_only, (p + 63) // 64 * 64)
    _check(lib, n, p, K, hi_only, (p + 7) // 8 * 8 + 8)


@pytest.mark.parametrize("hi_only,n", [(False, 70001), (True, 140001)])
def test_x_beyond_the_memory_side_cache(lib, hi_only, n):
    _check(lib, n, 1000, 10, hi_only, 1024, reps=3)


@pytest.mark.parametrize("many", [1, 30, 70])
@pytest.mark.parametrize("chains,K", [(4, 16), (2, 16), (2, 32), (1, 64), (1, 20), (1, 5)])
def test_batched_rows_off_cache_lines(lib, chains, K, many):
    """Every chain of a batch equals the oracle's gradient to the form's bar, rows off lines; the
    batch repeated until its gradient workgroups take 64, 128 and 256 columns."""
    import torch
    rng = np.random.default_rng([chains, K])
    probs, Bs, want = [], [], []
    for n, p in ((130, 65), (3000, 200), (64, 31)):
        X = torch.from_numpy(rng.normal(size=(n, p)).astype(np.float32)).cuda()
        y = rng.integers(0, K, size=n).astype(np.int32)
        hi = torch.full((n, (p + 7) // 8 * 8), float("nan"), dtype=torch.bfloat16, device="cuda")
        lo = torch.full_like(hi, float("nan"))
        hi[:, :p] = X.to(torch.bfloat16)
        lo[:, :p] = (X - hi[:, :p].float()).to(torch.bfloat16)
        probs.append(lib.Problem(hi[:, :p], torch.from_numpy(y).cuda(), K, X_lo=lo[:, :p]))
        B = rng.normal(0.0, 0.5 / np.sqrt(p), size=(chains, p, K)).astype(np.float32)
        Bs.append(torch.from_numpy(B).cuda())
        Xe = (hi[:, :p].double() + lo[:, :p].double()).cpu().numpy()
        B64 = B.astype(np.float64)
        B64[:, :, -1] = 0.0
        want.append([oracle.log_kernel_and_grad(Xe, y, b) for b in B64])
    batch = lib.Batch(probs[:1] * many + probs[1:], chains=chains)
    _, G, logk = batch.zeros_state()
    batch.logpost_grad(Bs[:1] * many + Bs[1:], G, logk)
    torch.cuda.synchronize()
    G, logk = G[many - 1:], logk[many - 1:]
    for b, per in enumerate(want):
        for c, (lk, Go) in enumerate(per):
            g = G[b][c].double().cpu().numpy()
            assert np.linalg.norm(g - Go) / np.linalg.norm(Go) <= GTOL
            assert abs(float(logk[b, c]) - lk) <= 1e-4 * abs(lk)
