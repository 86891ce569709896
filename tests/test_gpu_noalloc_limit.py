"""hmc_logpost_grad_noalloc at the limit of its built-in workspace (GPU tier): wide-p problems whose
workspace lies within a few KB of 32 MiB, with a partial last 16-row tile, and split planes that
fill it exactly are taken, with the workspace call's bits."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p,K,dtype,pin", [(107, 15788, 50, "float64", True), (778, 6919, 62, "float64", False),
                                             (1538, 4843, 64, "float64", False), (4342, 37913, 26, "float32", False),
                                             (267992, 17589, 12, "bfloat16", False)])
def test_problems_at_the_limit(lib, n, p, K, dtype, pin):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    ldx = (p + 7) // 8 * 8 if dtype == "bfloat16" else p
    X = torch.empty(n, ldx, device="cuda", dtype=getattr(torch, dtype)).normal_(0.0, 1.0, generator=g)[:, :p]
    y = torch.randint(0, K, (n,), generator=g, device="cuda", dtype=torch.int32)
    prob = lib.Problem(X, y, K, pin_last_class=pin)
    assert abs(lib.hmc_workspace_bytes(prob.desc) - (32 << 20)) <= 16 << 10
    B = (0.01 * torch.randn(p, K, generator=g, device="cuda", dtype=prob.dtype)).contiguous()
    if pin:
        B[:, -1] = 0.0
    want, Gw = lib.logpost_grad(prob, B)
    logk, G = torch.empty_like(want), torch.empty_like(B)
    lib.hmc_logpost_grad_noalloc(prob.desc, B, logk, G)
    assert float(logk) == float(want) and bool((G == Gw).all())
    del prob, X
    torch.cuda.empty_cache()
