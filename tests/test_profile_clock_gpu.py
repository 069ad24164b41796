"""tlora_profile_clock names the most recent product that took a sample: the pair of a block among them, and none after a call
without one."""
import pytest

pytestmark = pytest.mark.gpu


def _layer(torch, d_in, d_out, tokens):
    from paper_2602_07263_amd import tlora
    rnd = lambda *s: torch.randn(*s, device="cuda").to(torch.bfloat16)
    lp = tlora.LayerProblem("bf16", d_in, d_out, [8], [0, tokens], [1.0], rnd(tokens, d_in), rnd(d_in, d_out), [rnd(d_in, 8)], [rnd(8, d_out)])
    return lp, rnd(tokens, d_out)


def test_clock_of_pairs_and_of_calls_without_a_sample():
    import torch
    from paper_2602_07263_amd import tlora
    d, dff, T = 1024, 2816, 300
    rnd = lambda *s: torch.randn(*s, device="cuda").to(torch.bfloat16)
    layers = {n: (rnd(i, o), [rnd(i, 8)], [rnd(8, o)]) for n, (i, o) in dict(gate=(d, dff), up=(d, dff), down=(dff, d)).items()}
    X = rnd(T, d)
    block = tlora.MlpBlock("bf16", d, dff, [8], [0, T], [1.0], X, rnd(d), 1e-5, layers)
    Out, dX, grads = torch.empty_like(X), torch.empty_like(X), block.new_grads()
    general, dYg = _layer(torch, 1024, 1024, 300)
    small, dYs = _layer(torch, 1024, 1024, 16)
    try:
        tlora.tlora_profile(1)
        block.fwd(Out)
        block.bwd(rnd(T, d), dX, grads)                 # its last product is the pair's
        fwd, bwd = tlora.tlora_profile_clock()
        assert 0.1 < fwd < 4.0 and 0.1 < bwd < 4.0, (fwd, bwd)
        for lp, dY, sampled in ((general, dYg, True), (small, dYs, False), (general, dYg, True)):
            Y, dx, dA, dB = lp.new_outputs()
            lp.fwd(Y)
            lp.bwd(dY, dx, dA, dB, reuse_S=True)
            fwd, bwd = tlora.tlora_profile_clock()
            assert (fwd > 0.1 and bwd > 0.1) if sampled else (fwd, bwd) == (0.0, 0.0), (lp.T, fwd, bwd)
    finally:
        tlora.tlora_profile(0)
