"""The calls that this library is used for, as cases that can be timed and checked.

A case names a kind of call, a storage form of X and the sizes; `prepare` makes what a
program holds before the call (X on the GPU, labels, coefficients, the problem with its
workspace, a plan), `run` makes one pass through the public entry points and returns what
it computes, `exact` gives the same values in float64 without the library, and `work` the
bytes and operations a pass cannot do without.

Kinds:
  grad      logpost_grad: log K(B) and its gradient (the unit of all the others)
  autograd  LogPosterior.apply forward and backward
  leapfrog  L leapfrog updates in place, launched one by one
  sample    HMC transitions launched one by one, all records kept
  plan      one HMC transition as a captured graph, replayed
  batch     transitions of four (or fewer) chains of many uneven problems
  predict   posterior-predictive classification over coefficient samples
  split     encoding of X as bfloat16 planes

Forms: f64, f32, bf16x2 (hi + lo planes), bf16 (hi plane alone).
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_1402_4089_amd as hmc

LINKS = {"softmax": hmc.HMC_LINK_SOFTMAX, "poisson": hmc.HMC_LINK_POISSON, "probit": hmc.HMC_LINK_PROBIT}
PRIORS = {"gauss": hmc.HMC_PRIOR_GAUSS, "cauchy": hmc.HMC_PRIOR_CAUCHY}
X_BYTES = {"f64": 8, "f32": 4, "bf16x2": 4, "bf16": 2}
PLAN_SLOTS = 1 << 20          # iterations a plan's records hold
PHILOX_SEED = 1234


def listed():
    return [
        # the smallest problem of the benchmark: a single call, where launches and latency count
        dict(name="grad_small_f64", kind="grad", form="f64", n=500, p=20, K=3),
        # the same problem inside a sampling run: one replayed transition of ten updates
        dict(name="plan_small_f64", kind="plan", form="f64", n=500, p=20, K=3, L=10, step=0.5),
        # the default benchmark workload: one replayed transition of fifty updates
        dict(name="plan_f32", kind="plan", form="f32", n=20000, p=1000, K=10, L=50, step=0.35),
        # the MNIST-shaped run: pixels in [0, 1) and an intercept, a Cauchy prior, eager updates
        dict(name="leapfrog_mnist_f32", kind="leapfrog", form="f32", n=60000, p=785, K=10, L=10,
             step=0.2, prior="cauchy", pixels=True),
        # a torch program that differentiates log K: double precision, odd sizes, two class blocks
        dict(name="autograd_f64", kind="autograd", form="f64", n=5003, p=301, K=20, pin=False),
        # count regression, one coefficient column
        dict(name="grad_poisson_f32", kind="grad", form="f32", n=20000, p=1000, K=1, link="poisson"),
        # many more predictors than rows
        dict(name="leapfrog_widep_f32", kind="leapfrog", form="f32", n=2000, p=50000, K=4, L=10,
             step=0.1, scale=0.1),
        # the largest single problem: split-precision planes, 64 classes
        dict(name="grad_bf16x2", kind="grad", form="bf16x2", n=200000, p=4096, K=64),
        # eager sampling on the hi plane alone, odd sizes
        dict(name="sample_bf16", kind="sample", form="bf16", n=30011, p=1531, K=23, L=5, iters=2, step=0.3),
        # many uneven problems, four chains each, one replayed transition of twenty updates
        dict(name="batch_bf16x2", kind="batch", form="bf16x2", problems=16, sizes=5, chains=4, L=20, step=0.4,
             graph=True),
        # classes of held-out rows from one hundred recorded samples
        dict(name="predict_f32", kind="predict", form="f32", n=10000, p=785, K=10, S=100),
        # the one-time encoding of a large X
        dict(name="split_f32", kind="split", form="f32", n=50000, p=4096, lo=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _classes(rng):
    return rng.randint(2, 16) if rng.random() < 0.7 else rng.randint(17, 64)


def _sizes(rng, elements, n=(100, 200000), p=(4, 50000)):
    """n and p over the logarithm of their ranges, n p at most `elements`."""
    while True:
        a, b = _log_int(rng, *n), _log_int(rng, *p)
        if a * b <= elements:
            return a, b


def draw(rng):
    """A case of the same ranges: row counts from 100 to 200,000, 4 to 50,000 predictors, 2 to
    64 classes, every form, prior and link, rows with and without padding."""
    kind = rng.choice(["grad", "grad", "autograd", "leapfrog", "leapfrog", "sample", "plan", "plan",
                       "batch", "batch", "predict", "predict", "split"])
    if kind == "predict":
        f64 = rng.random() < 0.3
        while True:
            n, p, K, S = _log_int(rng, 500, 20000), _log_int(rng, 10, 1500), rng.randint(2, 20), _log_int(rng, 10, 200)
            if 16 * p + p * K <= 160 * 1024 // (8 if f64 else 4) and n * p * K * S <= (4 if f64 else 8) * 10 ** 9:
                return dict(kind=kind, form="f64" if f64 else "f32", n=n, p=p, K=K, S=S)
    if kind == "split":
        n, p = _sizes(rng, 2 * 10 ** 8, n=(1000, 200000), p=(16, 8192))
        return dict(kind=kind, form=rng.choice(["f32", "f32", "f64"]), n=n, p=p, lo=rng.random() < 0.7)
    if kind == "batch":
        while True:
            c = dict(kind=kind, form=rng.choice(["bf16x2", "bf16"]), problems=rng.randint(2, 16),
                     sizes=rng.randrange(10 ** 6), chains=rng.choice([1, 2, 4]), L=rng.randint(2, 20),
                     step=0.4, graph=rng.random() < 0.5)
            if work(c)["bytes"] <= 3e10 and work(c)["flops"] <= 1e12:
                return c
    form = rng.choice(["f64", "f32", "f32"] if kind == "autograd" else ["f64", "f32", "f32", "bf16x2", "bf16"])
    n, p = _sizes(rng, {"f64": 4 * 10 ** 7, "f32": 10 ** 8, "bf16x2": 4 * 10 ** 8, "bf16": 4 * 10 ** 8}[form])
    c = dict(kind=kind, form=form, n=n, p=p, K=_classes(rng), prior=rng.choice(["gauss", "cauchy"]),
             pin=rng.random() < 0.7)
    if form in ("f64", "f32"):
        c["pad"] = rng.choice([0, 0, 0, rng.randint(1, 64)])
    if kind == "grad" and form in ("f64", "f32") and rng.random() < 0.4:
        c.update(K=1, link=rng.choice(["poisson", "probit"]), pin=False)
    if kind in ("leapfrog", "plan", "sample"):
        most = max(1, 4 * 10 ** 9 // (n * p * X_BYTES[form]))
        c.update(L=rng.randint(1, max(1, min(20, most))), step=0.1)
    if kind == "sample":
        c.update(iters=rng.randint(1, 3))
    return c


# ---------------------------------------------------------------- inputs, from the seed alone

def _gen(seed, extra=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + extra)
    return g


def _normal(g, *shape, dtype=torch.float64):
    return torch.randn(*shape, generator=g, device="cuda", dtype=dtype)


def _make_x(case, n, p, g):
    """X in float64 or float32 (the type the planes are split from is float32)."""
    dtype = torch.float64 if case["form"] == "f64" else torch.float32
    pad = case.get("pad", 0)
    X = torch.empty(n, p + pad, device="cuda", dtype=dtype)
    if case.get("pixels"):
        X.uniform_(0.0, 1.0, generator=g)
        X[:, p - 1] = 1.0
    else:
        X.normal_(0.0, 1.0, generator=g)
    return X[:, :p]


def _truth(case, p, K, g):
    B = _normal(g, p, K) * (0.1 if case.get("pixels") else 0.5 if case.get("link") else 1.0) / (
        1.0 if case.get("pixels") else math.sqrt(p))
    if case.get("pin", True) and not case.get("link"):
        B -= B[:, -1:].clone()
    return B


def _times(X, B):
    """X B in X's type, in row blocks."""
    out = torch.empty(X.shape[0], B.shape[1], device="cuda", dtype=torch.float64)
    rows = max(1, (1 << 27) // X.shape[1])
    for i in range(0, X.shape[0], rows):
        out[i:i + rows] = (X[i:i + rows] @ B.to(X.dtype)).double()
    return out


def _labels(case, X, Bt, g):
    """Labels drawn from the model at the generating coefficients."""
    Z = _times(X, Bt)
    if case.get("link") == "poisson":
        return torch.poisson(Z[:, 0].exp(), generator=g).to(torch.int32)
    if case.get("link") == "probit":
        return (Z[:, 0] + _normal(g, Z.shape[0]) > 0).to(torch.int32)
    u = torch.rand(Z.shape, generator=g, device="cuda", dtype=torch.float64).clamp_min(1e-300)
    return (Z - (-u.log()).log()).argmax(1).to(torch.int32)


def _state(Bt, dtype, g, chains=None):
    """A point on the way of a chain: the generating coefficients, shrunk, and some noise."""
    shape = Bt.shape if chains is None else (chains,) + tuple(Bt.shape)
    B = 0.5 * Bt + 0.1 * Bt.std() * _normal(g, *shape)
    B = torch.where(Bt == 0, 0.0, B)               # the pinned column
    return B.to(dtype).contiguous()


def _batch_sizes(case):
    """Uneven problems: n ~ U[1k, 50k], p ~ U[64, 2048], K ~ U[2, 16]."""
    r = random.Random(case["sizes"])
    return [(r.randint(1000, 50000), r.randint(64, 2048), r.randint(2, 16)) for _ in range(case["problems"])]


def _state_dtype(case):
    return torch.float64 if case["form"] == "f64" else torch.float32


def _inputs(case, seed, n=None, p=None, K=None, extra=0, chains=None):
    n, p, K = n or case["n"], p or case["p"], K or case["K"]
    g = _gen(seed, extra)
    X = _make_x(case, n, p, g)
    Bt = _truth(case, p, K, g)
    y = _labels(case, X, Bt, g)
    return X, y, _state(Bt, _state_dtype(case), g, chains), g


def _eps(case, n, p):
    """Step size as a share of 1 / (the largest singular value of X, estimated by its law)."""
    top = math.sqrt(0.25 * n * p) if case.get("pixels") else math.sqrt(n) + math.sqrt(p)
    return case["step"] / top


def _planes(case, X):
    """(operand, lo plane) of the form: the matrix itself, or its encoding."""
    if case["form"] in ("f64", "f32"):
        return X, None
    return hmc.split_bf16(X, hi_only=case["form"] == "bf16")


def _problem(case, X, y, K):
    Xd, lo = _planes(case, X)
    return hmc.Problem(Xd, y, K, PRIORS[case.get("prior", "gauss")], case.get("scale", 1.0),
                       case.get("pin", True) and "link" not in case, X_lo=lo,
                       link=LINKS[case.get("link", "softmax")])


# ---------------------------------------------------------------- what a program has in hand

def prepare(case, seed):
    kind = case["kind"]
    if kind == "split":
        return dict(case=case, X=_make_x(case, case["n"], case["p"], _gen(seed)))
    if kind == "predict":
        g = _gen(seed)
        return dict(case=case, X=_make_x(case, case["n"], case["p"], g), samples=_samples(case, g))
    if kind == "batch":
        return _prepare_batch(case, seed)
    X, y, B, g = _inputs(case, seed)
    prob = _problem(case, X, y, case["K"])
    st = dict(case=case, prob=prob, B=B)
    if kind == "autograd":
        st["B"] = B.requires_grad_()
    if kind in ("leapfrog", "sample", "plan"):
        st["eps"] = _eps(case, case["n"], case["p"])
        st["logk"], st["G"] = hmc.logpost_grad(prob, B)
    if kind == "leapfrog":
        st["eta"] = _momentum(case, g)
    if kind == "plan":
        st["plan"], st["records"] = hmc.plan(prob, B, st["G"], st["logk"], st["eps"], case["L"], PLAN_SLOTS,
                                             seed=PHILOX_SEED + seed, record_samples=False)
    st["seed"] = PHILOX_SEED + seed
    return st


def _momentum(case, g):
    eta = _normal(g, case["p"], case["K"])
    if case.get("pin", True):
        eta[:, -1] = 0.0
    return eta.to(_state_dtype(case)).contiguous()


def _samples(case, g):
    """Recorded draws around a common point, the last class pinned."""
    Bt = _truth(case, case["p"], case["K"], g)
    S = Bt + 0.3 * _normal(g, case["S"], case["p"], case["K"]) / math.sqrt(case["p"])
    S[:, :, -1] = 0.0
    return S.to(_state_dtype(case)).contiguous()


def _prepare_batch(case, seed):
    probs, B = [], []
    for b, (n, p, K) in enumerate(_batch_sizes(case)):
        X, y, Bb, _ = _inputs(case, seed, n, p, K, extra=b + 1, chains=case["chains"])
        probs.append(_problem(case, X, y, K))
        B.append(Bb)
    batch = hmc.Batch(probs, chains=case["chains"])
    _, G, logk = batch.zeros_state()
    batch.logpost_grad(B, G, logk)
    st = dict(case=case, batch=batch, B=B, G=G, logk=logk, seed=PHILOX_SEED + seed,
              eps=[_eps(case, n, p) for n, p, _ in _batch_sizes(case)])
    if case["graph"]:
        st["plan"], st["records"] = batch.plan(B, G, logk, st["eps"], case["L"], PLAN_SLOTS // 64, seed=st["seed"],
                                               records=False)
    return st


# ---------------------------------------------------------------- one pass

def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "grad":
        return hmc.logpost_grad(st["prob"], st["B"])
    if kind == "autograd":
        B = st["B"]
        B.grad = None
        logk = hmc.LogPosterior.apply(B, st["prob"])
        logk.backward()
        return logk.detach(), B.grad
    if kind == "leapfrog":
        hmc.leapfrog(st["prob"], st["B"], st["eta"], st["G"], st["logk"], st["eps"], case["L"])
        return st["B"], st["eta"], st["G"], st["logk"]
    if kind == "sample":
        rec = hmc.sample(st["prob"], st["B"], st["G"], st["logk"], st["eps"], case["L"], case["iters"],
                         seed=st["seed"])
        return st["B"], st["G"], st["logk"], rec
    if kind == "plan":
        st["plan"].launch(1)
        return st["B"], st["G"], st["logk"]
    if kind == "batch":
        if case["graph"]:
            st["plan"].launch(1)
            return st["B"], st["G"], st["logk"]
        rec = st["batch"].sample(st["B"], st["G"], st["logk"], st["eps"], case["L"], 1, seed=st["seed"])
        return st["B"], st["G"], st["logk"], rec
    if kind == "predict":
        return hmc.posterior_predictive(st["X"], st["samples"], case["K"])
    return hmc.split_bf16(st["X"], hi_only=not case["lo"])


# ---------------------------------------------------------------- bytes and operations

def work(case):
    kind = case["kind"]
    if kind == "split":
        s, n, p = X_BYTES[case["form"]], case["n"], case["p"]
        return {"bytes": n * p * (s + (4 if case["lo"] else 2)), "flops": 0}
    if kind == "predict":
        s, n, p, K, S = X_BYTES[case["form"]], case["n"], case["p"], case["K"], case["S"]
        return {"bytes": n * p * s + S * p * K * s + n * K * 8 + n * 4, "flops": 2 * n * p * (K - 1) * S}
    if kind == "batch":
        per = [_gradient(case, n, p, K, case["chains"]) for n, p, K in _batch_sizes(case)]
        evals = case["L"]
    else:
        per = [_gradient(case, case["n"], case["p"], case["K"], 1)]
        evals = case.get("L", 1) * case.get("iters", 1)
    return {"bytes": evals * sum(b for b, _ in per), "flops": evals * sum(f for _, f in per)}


def _gradient(case, n, p, K, chains):
    """Bytes and operations of one gradient evaluation: X and labels read, coefficients read,
    gradient written; two contractions over the free classes."""
    s = 8 if case["form"] == "f64" else 4
    free = K - 1 if case.get("pin", True) and "link" not in case else K
    return n * p * X_BYTES[case["form"]] + 4 * n + 2 * chains * p * K * s, 4 * n * p * free * chains


# ---------------------------------------------------------------- the same in 64 bits

def _exact_x(case, X):
    """The row blocks of the values the device sees, in float64."""
    rows = max(1, (1 << 27) // X.shape[1])
    for i in range(0, X.shape[0], rows):
        x = X[i:i + rows]
        if case["form"] in ("f64", "f32"):
            x = x.double()
        else:
            hi = x.bfloat16()
            lo = (x - hi.float()).bfloat16().double() if case["form"] == "bf16x2" else 0.0
            x = hi.double() + lo
        yield slice(i, i + rows), x


def _exact_grad(case, X, y, B):
    """log K and gradient at B, in float64."""
    link = case.get("link", "softmax")
    pin = case.get("pin", True) and link == "softmax"
    mask = torch.ones_like(B)
    if pin:
        mask[:, -1] = 0.0
    B = B * mask
    logk, G = torch.zeros((), dtype=torch.float64, device="cuda"), torch.zeros_like(B)
    for at, x in _exact_x(case, X):
        z, yy = x @ B, y[at].long()
        if link == "poisson":
            mu = z[:, 0].exp()
            logk += (yy * z[:, 0] - mu).sum()
            r = (yy - mu)[:, None]
        elif link == "probit":
            s = torch.where(yy == 1, 1.0, -1.0).double()
            w = s * z[:, 0]
            lp = torch.special.log_ndtr(w)
            logk += lp.sum()
            r = (s * torch.exp(-0.5 * w * w - 0.5 * math.log(2.0 * math.pi) - lp))[:, None]
        else:
            ls = torch.log_softmax(z, 1)
            logk += ls.gather(1, yy[:, None]).sum()
            r = -ls.exp()
            r.scatter_add_(1, yy[:, None], torch.ones_like(r[:, :1]))
        G += x.T @ r
    s = case.get("scale", 1.0)
    if case.get("prior", "gauss") == "cauchy":
        logk -= (torch.log1p((B / s) ** 2) * mask).sum()
        G -= 2.0 * B / (s * s + B * B)
    else:
        logk -= (B * B * mask).sum() / (2.0 * s * s)
        G -= B / (s * s)
    return logk, G * mask


def _philox(words, key):
    """Philox4x32-10 on four arrays of 32-bit words."""
    c, low = [np.asarray(w, dtype=np.uint64) for w in words], np.uint64(0xFFFFFFFF)
    k = [np.uint64(key & 0xFFFFFFFF), np.uint64((key >> 32) & 0xFFFFFFFF)]
    for r in range(10):
        if r:
            k = [(k[0] + np.uint64(0x9E3779B9)) & low, (k[1] + np.uint64(0xBB67AE85)) & low]
        a, b = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(b >> np.uint64(32)) ^ c[1] ^ k[0], b & low, (a >> np.uint64(32)) ^ c[3] ^ k[1], a & low]
    return c


def _u53(hi, lo):
    return ((((hi << np.uint64(32)) | lo) >> np.uint64(11)).astype(np.float64) + 0.5) * 2.0 ** -53


def _draws(seed, chain, it, count):
    """(standard normals, uniform) of one transition of a chain."""
    e = np.arange((count + 1) // 2, dtype=np.uint64)
    c = _philox([e, np.full_like(e, it), np.full_like(e, chain), np.zeros_like(e)], seed)
    r, a = np.sqrt(-2.0 * np.log(_u53(c[0], c[1]))), 2.0 * np.pi * _u53(c[2], c[3])
    xi = np.stack([r * np.cos(a), r * np.sin(a)], 1).reshape(-1)[:count]
    u = _philox([np.zeros(1), np.full(1, it), np.full(1, chain), np.ones(1)], seed)
    return torch.from_numpy(xi).cuda(), float(_u53(u[0], u[1])[0])


def _exact_leapfrog(case, X, y, B, eta, G, eps, L):
    logk = None
    for _ in range(L):
        eta = eta + 0.5 * eps * G
        B = B + eps * eta
        logk, G = _exact_grad(case, X, y, B)
        eta = eta + 0.5 * eps * G
    return B, eta, G, logk


def _exact_chain(case, X, y, B, eps, L, iters, seed, chain):
    """iters transitions of one chain: (B, G, logk, records)."""
    logk, G = _exact_grad(case, X, y, B)
    H, acc, div, states = [], [], [], []
    for t in range(iters):
        xi, u = _draws(seed, chain, t, B.numel())
        eta = xi.reshape(B.shape).clone()
        if case.get("pin", True):
            eta[:, -1] = 0.0
        Bn, en, Gn, ln = _exact_leapfrog(case, X, y, B, eta, G, eps, L)
        h0, h1 = float(-logk + 0.5 * (eta * eta).sum()), float(-ln + 0.5 * (en * en).sum())
        ok = math.isfinite(h1) and math.log(u) < h0 - h1
        if ok:
            B, G, logk = Bn, Gn, ln
        H.append([h0, h1])
        acc.append(int(ok))
        div.append(int(not math.isfinite(h1) or h1 - h0 > 1000.0))
        states.append(B)
    whole = dict(dtype=torch.int32, device="cuda")
    return B, G, logk, dict(accepted=torch.tensor(acc, **whole), divergent=torch.tensor(div, **whole),
                            H=torch.tensor(H, dtype=torch.float64, device="cuda"), samples=torch.stack(states))


def exact(case, seed):
    kind = case["kind"]
    if kind == "split":
        X = _make_x(case, case["n"], case["p"], _gen(seed)).double()
        hi = X.to(torch.bfloat16).double()       # torch rounds a float64 through float32: within the type's bound
        return hi, ((X - hi).to(torch.bfloat16).double() if case["lo"] else None)
    if kind == "predict":
        return _exact_predict(case, seed)
    if kind == "batch":
        return _exact_batch(case, seed)
    X, y, B, g = _inputs(case, seed)
    B = B.double()
    if kind in ("grad", "autograd"):
        return _exact_grad(case, X, y, B)
    eps = _eps(case, case["n"], case["p"])
    if kind == "leapfrog":
        eta = _momentum(case, g).double()
        return _exact_leapfrog(case, X, y, B, eta, _exact_grad(case, X, y, B)[1], eps, case["L"])
    out = _exact_chain(case, X, y, B, eps, case["L"], case.get("iters", 1), PHILOX_SEED + seed, 0)
    return out if kind == "sample" else out[:3]


def _exact_predict(case, seed):
    g = _gen(seed)
    X = _make_x(case, case["n"], case["p"], g).double()
    mean = torch.zeros(case["n"], case["K"], dtype=torch.float64, device="cuda")
    for B in _samples(case, g).double():
        mean += torch.softmax(X @ B, 1)
    mean /= case["S"]
    return mean, mean.argmax(1).to(torch.int32)


def _exact_batch(case, seed):
    C = case["chains"]
    B, G, logk, acc, div, H = [], [], [], [], [], []
    for b, (n, p, K) in enumerate(_batch_sizes(case)):
        X, y, B0, _ = _inputs(case, seed, n, p, K, extra=b + 1, chains=C)
        got = [_exact_chain(case, X, y, B0[c].double(), _eps(case, n, p), case["L"], 1, PHILOX_SEED + seed, b * C + c)
               for c in range(C)]
        B.append(torch.stack([o[0] for o in got]))
        G.append(torch.stack([o[1] for o in got]))
        logk.append(torch.stack([o[2] for o in got]))
        acc += [o[3]["accepted"] for o in got]
        div += [o[3]["divergent"] for o in got]
        H += [o[3]["H"] for o in got]
    logk = torch.stack(logk)
    if case["graph"]:
        return B, G, logk
    return B, G, logk, dict(accepted=torch.stack(acc, 1), divergent=torch.stack(div, 1), H=torch.stack(H, 1))
