"""Small problems in one workgroup (GPU tier): gradient, leapfrog, transitions and plans at the
edges of its range (one row, one predictor, one class column, 512 / 513 / 1024 rows, 16-column
blocks with remainders, 4, 8 and 16 padded classes), padded rows, both precisions, priors, links.

Against the oracle (the bars of the general path) and against the general path, which an explicit
tuning selects. FP32 logits and softmax are formed alike in both, so log K may differ only by the
order of a float64 sum: relative 1e-12."""
import numpy as np
import pytest

import oracle
from workloads import make_draws

pytestmark = pytest.mark.gpu

SHAPES = [  # n, p, K, pinned, row padding
    (1, 1, 2, True, 0), (3, 17, 4, True, 2), (64, 16, 5, False, 0), (100, 33, 8, True, 0), (500, 20, 3, True, 0),
    (511, 4, 9, True, 1), (512, 8, 16, False, 0), (513, 31, 4, True, 0), (1024, 10, 6, True, 3), (37, 250, 7, True, 0),
    (15, 256, 16, True, 0), (129, 127, 4, False, 1), (1000, 2, 2, True, 0),
]


def _case(n, p, K, pin, pad, dtype, link=0):
    import torch
    rng = np.random.default_rng([n, p, K])
    X = rng.normal(size=(n, p)).astype(dtype)
    y = (rng.poisson(1.0, n) if link == 1 else rng.integers(0, max(K, 2), n)).astype(np.int32)
    B = rng.normal(0.0, 0.5 / np.sqrt(p), size=(p, K)).astype(dtype)
    if pin:
        B[:, -1] = 0.0
    buf = torch.full((n, p + pad), float("nan"), dtype=torch.from_numpy(X).dtype, device="cuda")
    buf[:, :p] = torch.from_numpy(X).cuda()
    return X.astype(np.float64), y, B, buf[:, :p], torch.from_numpy(y).cuda()


def _general(lib, prob):
    """The same problem on the general row-tile path (an explicit variant that covers p)."""
    w = 16 if prob.dtype.itemsize == 4 and prob.p > 128 else 8
    return dict(path=1, waves=w, mb=1 if prob.p <= 16 * w else 2, grid=0, rows_per_slice=0)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("prior", [oracle.GAUSS, oracle.CAUCHY])
@pytest.mark.parametrize("n,p,K,pin,pad", SHAPES)
def test_gradient(lib, n, p, K, pin, pad, prior, dtype):
    import torch
    X, y, B, Xd, yd = _case(n, p, K, pin, pad, dtype)
    prob = lib.Problem(Xd, yd, K, prior, 0.7, pin)
    gen = lib.Problem(Xd, yd, K, prior, 0.7, pin, tuning=_general(lib, prob))
    Bd = torch.from_numpy(B).cuda()
    logk, G = lib.logpost_grad(prob, Bd)
    lg, Gg = lib.logpost_grad(gen, Bd)
    lk, Go = oracle.log_kernel_and_grad(X, y, B.astype(np.float64), prior, 0.7, int(pin))
    tol = 1e-12 if dtype == np.float64 else 1e-5
    assert abs(float(logk) - float(lg)) <= 1e-12 * abs(lk)
    for g in (G, Gg):
        assert np.linalg.norm(g.double().cpu().numpy() - Go) <= tol * max(np.linalg.norm(Go), 1e-3)
    assert abs(float(logk) - lk) <= tol * max(abs(lk), 1.0)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("link", [1, 2])
@pytest.mark.parametrize("n,p", [(1, 1), (400, 20), (777, 33), (1024, 64)])
def test_links(lib, n, p, link, dtype):
    import torch
    X, y, B, Xd, yd = _case(n, p, 1, False, 1, dtype, link)
    prob = lib.Problem(Xd, yd, 1, 0, 1.0, False, link=link)
    logk, G = lib.logpost_grad(prob, torch.from_numpy(B).cuda())
    lk, Go = oracle.log_kernel_and_grad(X, y, B.astype(np.float64), 0, 1.0, 0, link)
    tol = 1e-11 if dtype == np.float64 else 1e-5
    assert np.linalg.norm(G.double().cpu().numpy() - Go) <= tol * max(np.linalg.norm(Go), 1e-3)
    assert abs(float(logk) - lk) <= tol * max(abs(lk), 1.0)


@pytest.mark.parametrize("n,p,K,pin,pad", SHAPES)
def test_transitions_leapfrog_and_plan(lib, n, p, K, pin, pad):
    """FP64: replayed transitions equal the oracle chain, eagerly and as a plan launched in two
    parts with other work between; a leapfrog run equals the oracle's."""
    import torch
    X, y, B, Xd, yd = _case(n, p, K, pin, pad, np.float64)
    prob = lib.Problem(Xd, yd, K, 0, 1.0, pin)
    eps, L, T = 0.3 / (np.sqrt(n) + np.sqrt(p)), 4, 6
    d = make_draws(p, K, T, seed=(n, p, K))
    xi, u = torch.from_numpy(d.xi).cuda(), torch.from_numpy(d.u).cuda()
    orc = oracle.sample(X, y, K, d.xi, d.u, eps, L, pin_last_class=int(pin), B0=B)
    for graph in (False, True):
        Bd = torch.from_numpy(B).cuda()
        logk, G = lib.logpost_grad(prob, Bd)
        if graph:
            plan, out = lib.plan(prob, Bd, G, logk, eps, L, T, normals=xi, uniforms=u)
            plan.launch(2)
            torch.cuda.synchronize()
            torch.zeros(1000, device="cuda").add_(1)
            plan.launch(T - 2)
        else:
            out = lib.sample(prob, Bd, G, logk, eps, L, T, normals=xi, uniforms=u)
        torch.cuda.synchronize()
        assert np.array_equal(out["accepted"].cpu().numpy(), orc["accepted"])
        assert np.max(np.abs(out["samples"].cpu().numpy() - orc["samples"])) <= 1e-10
        assert np.max(np.abs(Bd.cpu().numpy() - orc["samples"][-1])) <= 1e-10
    Bd = torch.from_numpy(B).cuda()
    logk, G = lib.logpost_grad(prob, Bd)
    eta0 = d.xi[0] * oracle.free_mask(p, K, int(pin))
    eta = torch.from_numpy(eta0).cuda()
    lib.leapfrog(prob, Bd, eta, G, logk, eps, L)
    Bo, eo, Go, lk = oracle.leapfrog(X, y, B, eta0, oracle.grad_log_kernel(X, y, B, 0, 1.0, int(pin)), eps, L,
                                     pin_last_class=int(pin))
    for got, want in ((Bd, Bo), (eta, eo), (G, Go)):
        assert np.linalg.norm(got.cpu().numpy() - want) <= 1e-12 * max(np.linalg.norm(want), 1.0)
    assert abs(float(logk) - lk) <= 1e-12 * max(abs(lk), 1.0)
