"""Autotuning of small problems (GPU tier): where the built-in rule runs leapfrog updates in one
workgroup, tuning="auto" keeps it, also at sizes whose single gradient runs on the row tile with the
rule and with explicit tunings alike, so that gradient times alone cannot tell them apart."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n,p,K,pin", [
    (np.float32, 100, 64, 3, True), (np.float32, 513, 31, 4, True), (np.float32, 100, 33, 8, True),
    (np.float32, 300, 40, 4, True), (np.float64, 64, 16, 5, False), (np.float64, 500, 20, 3, True)])
def test_the_rule_is_kept(lib, tmp_path, monkeypatch, dtype, n, p, K, pin):
    import torch
    from paper_1402_4089_amd import tuning
    monkeypatch.setenv(tuning.ENV, str(tmp_path / "cache.json"))
    rng = np.random.default_rng([n, p, K])
    X = torch.from_numpy(rng.normal(size=(n, p)).astype(dtype)).cuda()
    y = torch.from_numpy(rng.integers(0, K, n).astype(np.int32)).cuda()
    prob = lib.Problem(X, y, K, pin_last_class=pin, tuning="auto")
    assert prob.tuning["path"] == 0 and prob.tuned_us > 0
    B = prob.zeros_state()
    logk, G = lib.logpost_grad(prob, B)
    eta = torch.zeros_like(B)
    prob.ws.fill_(0xA5)
    lib.leapfrog(prob, B, eta, G, logk, 1e-3, 3)
    assert bool((prob.ws == 0xA5).all())          # the one-workgroup form works in its LDS alone
