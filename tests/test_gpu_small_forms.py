"""The one-workgroup form of small problems over what its rule accepts (GPU tier): 1 to 16 padded
classes, 512 and 1024 threads, one row to 1024, in both precisions, for gradients, leapfrog runs,
transitions (replayed and Philox draws, annealed, divergent) and plans, against the FP64 oracle.
Every call is checked to have run there: that form leaves the problem's workspace alone but for a
plan's iteration counter."""
import numpy as np
import pytest

import oracle
from oracle import philox

pytestmark = pytest.mark.gpu

F64, F32 = np.float64, np.float32
# n, p, K, pinned, row padding
BOTH = [(1, 1, 2, True, 0), (3, 17, 4, True, 2), (500, 20, 3, True, 0), (1000, 2, 2, True, 1), (17, 33, 2, True, 0),
        (513, 2, 3, False, 0), (512, 3, 4, False, 3), (100, 5, 8, True, 0), (60, 3, 12, True, 1),
        (30, 7, 16, False, 0), (20, 8, 16, True, 0), (100, 2, 16, False, 0)]
GRADIENTS = [(dt, *s) for dt in (F64, F32) for s in BOTH] + [
    (F64, 1024, 3, 2, True, 0), (F64, 1024, 1, 3, True, 2), (F32, 64, 16, 5, False, 0), (F32, 513, 5, 4, False, 1),
    (F32, 90, 9, 16, False, 0), (F32, 120, 3, 16, True, 0), (F32, 90, 32, 5, True, 0), (F32, 129, 16, 9, True, 0)]
UPDATES = [(dt, *s) for dt in (F64, F32) for s in BOTH + [
    (1024, 3, 2, True, 0), (1024, 2, 4, True, 2), (511, 4, 9, True, 0), (33, 31, 7, True, 0), (16, 17, 10, True, 1),
    (64, 12, 12, False, 0), (50, 130, 2, True, 0), (1023, 15, 2, False, 1), (200, 17, 8, True, 0),
    (128, 33, 4, False, 0), (200, 3, 16, False, 0)]] + [
    (F64, 100, 120, 2, True, 0), (F32, 1024, 20, 3, True, 0), (F32, 700, 4, 9, True, 1), (F32, 33, 17, 16, False, 0)]


class Case:
    def __init__(self, lib, dtype, n, p, K, pin, pad, link=0, prior=oracle.GAUSS):
        import torch
        rng = np.random.default_rng([n, p, K])
        X = rng.normal(size=(n, p)).astype(dtype)
        self.y = (rng.poisson(1.0, n) if link == 1 else rng.integers(0, max(K, 2), n)).astype(np.int32)
        B = rng.normal(0.0, 0.5 / np.sqrt(p), size=(p, K)).astype(dtype)
        if pin:
            B[:, -1] = 0.0
        buf = torch.full((n, p + pad), float("nan"), dtype=torch.from_numpy(X).dtype, device="cuda")
        buf[:, :p] = torch.from_numpy(X).cuda()
        self.X, self.B, self.pin, self.link, self.prior = X.astype(F64), B.astype(F64), int(pin), link, prior
        self.Bd = torch.from_numpy(B).cuda()
        self.prob = lib.Problem(buf[:, :p], torch.from_numpy(self.y).cuda(), K, prior, 0.8, pin, link=link)
        self.eps = 0.3 / (np.sqrt(n) + np.sqrt(p))

    def state(self, lib):
        B = self.Bd.clone()
        logk, G = lib.logpost_grad(self.prob, B)
        self.prob.ws.fill_(0xA5)
        return B, logk, G

    def untouched(self, allowed=0):
        return int((self.prob.ws != 0xA5).sum()) <= allowed


def _close(got, want, rel, floor):
    got = got.double().cpu().numpy() if hasattr(got, "cpu") else np.asarray(got)
    assert np.linalg.norm(got - want) <= rel * max(float(np.linalg.norm(want)), floor)


@pytest.mark.parametrize("prior", [oracle.GAUSS, oracle.CAUCHY])
@pytest.mark.parametrize("dtype,n,p,K,pin,pad", GRADIENTS)
def test_gradient(lib, dtype, n, p, K, pin, pad, prior):
    c = Case(lib, dtype, n, p, K, pin, pad, prior=prior)
    c.prob.ws.fill_(0xA5)
    logk, G = lib.logpost_grad(c.prob, c.Bd)
    assert c.untouched()
    lk, Go = oracle.log_kernel_and_grad(c.X, c.y, c.B, prior, 0.8, c.pin)
    tol = 1e-12 if dtype == F64 else 1e-5
    _close(G, Go, tol, 1e-3)
    assert abs(float(logk) - lk) <= tol * max(abs(lk), 1.0)


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("link", [1, 2])
@pytest.mark.parametrize("n,p", [(1, 1), (400, 20), (777, 5), (1024, 2), (60, 40)])
def test_links(lib, n, p, link, dtype):
    c = Case(lib, dtype, n, p, 1, False, 1, link)
    c.prob.ws.fill_(0xA5)
    logk, G = lib.logpost_grad(c.prob, c.Bd)
    assert c.untouched()
    lk, Go = oracle.log_kernel_and_grad(c.X, c.y, c.B, 0, 0.8, 0, link)
    tol = 1e-11 if dtype == F64 else 1e-5
    _close(G, Go, tol, 1e-3)
    assert abs(float(logk) - lk) <= tol * max(abs(lk), 1.0)
    B, logk, G = c.state(lib)
    eta0 = np.random.default_rng(3).normal(size=(p, 1)).astype(dtype).astype(F64)
    import torch
    eta = torch.from_numpy(eta0.astype(dtype)).cuda()
    lib.leapfrog(c.prob, B, eta, G, logk, c.eps, 3)
    assert c.untouched()
    G0 = oracle.grad_log_kernel(c.X, c.y, c.B, 0, 0.8, 0, link)
    Bo, eo, Go, lk = oracle.leapfrog(c.X, c.y, c.B, eta0, G0, c.eps, 3, 0, 0.8, 0, link)
    for got, want in ((B, Bo), (eta, eo), (G, Go)):
        _close(got, want, 10 * tol, 1.0)
    assert abs(float(logk) - lk) <= 10 * tol * max(abs(lk), 1.0)


@pytest.mark.parametrize("dtype,n,p,K,pin,pad", UPDATES)
def test_leapfrog(lib, dtype, n, p, K, pin, pad):
    """Four updates: each adds a few roundings of the state and a gradient's error times eps."""
    import torch
    c = Case(lib, dtype, n, p, K, pin, pad, prior=oracle.CAUCHY)
    eta0 = np.random.default_rng([n, K]).normal(size=(p, K)).astype(dtype).astype(F64) * oracle.free_mask(p, K, c.pin)
    B, logk, G = c.state(lib)
    eta = torch.from_numpy(eta0.astype(dtype)).cuda()
    lib.leapfrog(c.prob, B, eta, G, logk, c.eps, 4)
    assert c.untouched()
    G0 = oracle.grad_log_kernel(c.X, c.y, c.B, oracle.CAUCHY, 0.8, c.pin)
    Bo, eo, Go, lk = oracle.leapfrog(c.X, c.y, c.B, eta0, G0, c.eps, 4, oracle.CAUCHY, 0.8, c.pin)
    tol = 1e-12 if dtype == F64 else 1e-5
    for got, want in ((B, Bo), (eta, eo), (G, Go)):
        _close(got, want, 4 * tol, 1.0)
    assert abs(float(logk) - lk) <= 4 * tol * max(abs(lk), 1.0)


@pytest.mark.parametrize("kind", ["replay", "philox", "annealed", "divergent"])
@pytest.mark.parametrize("dtype,n,p,K,pin,pad", UPDATES)
def test_transitions_and_plan(lib, dtype, n, p, K, pin, pad, kind):
    """Six transitions of four updates, launched singly and as a plan replayed in two parts: the
    oracle's decisions, flags, energies and states, and the plan's bits equal to the single calls'."""
    import torch
    c = Case(lib, dtype, n, p, K, pin, pad)
    T, L, seed, chain, first = 6, 4, 77, 3, 11
    eps = c.eps * (400.0 if kind == "divergent" else 1.0)
    if kind == "philox":
        xi, u = philox.draws(seed, chain, T, p, K, first_iter=first)
        draws = dict(seed=seed, chain=chain, first_iter=first)
    else:
        rng = np.random.default_rng([n, p, K, 5])
        xi, u = rng.standard_normal((T, p, K)), rng.uniform(1e-3, 1.0, T)
        draws = dict(normals=torch.from_numpy(xi).cuda(), uniforms=torch.from_numpy(u).cuda())
    temps = oracle.annealed_inv_temps(T, 50.0, 0.5) if kind == "annealed" else None
    if temps is not None:
        draws.update(inv_temperature=torch.from_numpy(temps).cuda())
    want = oracle.sample(c.X, c.y, K, xi, u, eps, L, 0, 0.8, c.pin, B0=c.B, inv_temps=temps)
    runs = []
    for graph in (False, True):
        B, logk, G = c.state(lib)
        if graph:
            plan, out = lib.plan(c.prob, B, G, logk, eps, L, T, **draws)
            plan.launch(2)
            torch.cuda.synchronize()
            torch.zeros(1000, device="cuda").add_(1)
            plan.launch(T - 2)
        else:
            out = lib.sample(c.prob, B, G, logk, eps, L, T, **draws)
        torch.cuda.synchronize()
        assert c.untouched(16 if graph else 0)
        runs.append((B, G, logk, out))
    for (B, G, logk, out) in runs:
        assert np.array_equal(out["accepted"].cpu().numpy(), want["accepted"])
        assert np.array_equal(out["divergent"].cpu().numpy(), want["divergent"])
        if kind == "divergent":
            continue                     # energies of runaway trajectories carry no common digits
        tol = 1e-10 if dtype == F64 else 1e-4
        assert np.max(np.abs(out["samples"].double().cpu().numpy() - want["samples"])) <= tol
        assert np.max(np.abs(B.double().cpu().numpy() - want["B"])) <= tol
        _close(G, want["G"], tol, 1.0)
        H = out["H"].cpu().numpy()
        assert np.max(np.abs(H - want["H"])) <= tol * max(1.0, float(np.max(np.abs(want["H"]))))
        assert abs(float(logk) - want["logk"]) <= tol * max(1.0, abs(want["logk"]))
    for a, b in zip(runs[0][:3], runs[1][:3]):
        assert torch.equal(a, b)
    for k in ("accepted", "divergent", "H", "samples"):
        assert torch.equal(runs[0][3][k], runs[1][3][k]) or kind == "divergent"
