"""More output tiles of idle jobs' gradients than a launch has work units: the reduction clears them."""
import pytest

pytestmark = pytest.mark.gpu


def test_gradients_of_tens_of_thousands_of_idle_jobs():
    import torch
    from paper_2602_07263_amd import tlora
    J, busy, d_in, d_out, scale = 32768, 1000, 8, 40960, 2.0
    g = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g).to(torch.bfloat16)
    X, W, dY = rnd(1, d_in), rnd(d_in, d_out), rnd(1, d_out)
    A, B, a, b = rnd(d_in, 1), rnd(1, d_out), rnd(d_in, 1), rnd(1, d_out)              # (the idle jobs share theirs)
    pick = lambda mine, idle: [idle] * busy + [mine] + [idle] * (J - busy - 1)
    nan = lambda *s: torch.full(s, float("nan"), device="cuda")
    dA, dB, da, db = nan(d_in, 1), nan(1, d_out), nan(d_in, 1), nan(1, d_out)
    lp = tlora.LayerProblem("bf16", d_in, d_out, [1] * J, [0] * (busy + 1) + [1] * (J - busy), [scale] * J, X, W, pick(A, a), pick(B, b))
    Y, dX = torch.empty_like(dY), torch.empty_like(X)
    try:
        lp.fwd(Y)
        lp.bwd(dY, dX, pick(dA, da), pick(dB, db), reuse_S=True)
        torch.cuda.synchronize()
    finally:
        tlora.tlora_set_option("plan_cache", 1)          # (the plan's tables are large)
    x, w, dy, A, B = (t.double() for t in (X, W, dY, A, B))
    # relative errors in the 2-norm: bf16 results and the bf16 S_j inside them 2^-9 / sqrt(3) each; S_j as two bf16 planes 2^-17
    for got, want, tol in ((Y, x @ w + scale * (x @ A) @ B, 4e-3), (dX, dy @ w.T + scale * (dy @ B.T) @ A.T, 4e-3),
                           (dA, scale * x.T @ (dy @ B.T), 2e-5), (dB, scale * (x @ A).T @ dy, 2e-5)):
        assert float((got.double() - want).norm() / want.norm()) <= tol
    assert not da.any() and not db.any()
