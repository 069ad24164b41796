"""Backbone products whose last row and column tiles are ragged: their lanes beyond the edge load nothing, or the next row of the
weight, so what the LDS held before (NaN here) must not reach a stored output."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tokens", [1, 9, 255, 257, 519])
@pytest.mark.parametrize("d_in,d_out", [(24, 32768), (160, 8), (96, 264), (256, 200), (1000, 544), (1024, 800)])
def test_ragged_edges(d_in, d_out, tokens):
    import torch
    from paper_2602_07263_amd import tlora
    g = torch.Generator(device="cuda").manual_seed(d_in + d_out + tokens)
    rnd = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).to(torch.bfloat16)
    layer = lambda X, W, A, B: tlora.LayerProblem("bf16", X.shape[1], W.shape[1], [4], [0, X.shape[0]], [2.0], X, W, [A], [B])
    nan = torch.full((16 * 256, 256), float("nan"), dtype=torch.bfloat16, device="cuda")     # 256 tiles: the LDS of every CU
    fill = layer(nan, nan[:256].repeat(1, 16), nan[:256, :4].contiguous(), nan[:4].repeat(1, 16))
    filled = fill.new_outputs()[0]
    X, dY = rnd(tokens, d_in), rnd(tokens, d_out)
    W, A, B = rnd(d_in, d_out, std=d_in ** -0.5), rnd(d_in, 4, std=d_in ** -0.5), rnd(4, d_out, std=0.05)
    lp = layer(X, W, A, B)
    Y, dX, _, _ = lp.new_outputs()
    Y.fill_(float("nan"))
    dX.fill_(float("nan"))
    fill.fwd(filled)
    lp.fwd(Y)
    fill.fwd(filled)
    lp.bwd(dY, dX, None, None, reuse_S=True)
    torch.cuda.synchronize()
    d = torch.float64
    M = W.to(d) + 2.0 * A.to(d) @ B.to(d)
    # one rounding to bf16 (2^-9 / sqrt(3) = 1.1e-3 in the 2-norm; an entry: 2^-9) and s_j S_j rounded once more, over a smaller part
    for got, want in ((Y, X.to(d) @ M), (dX, dY.to(d) @ M.T)):
        assert float((got.to(d) - want).norm() / want.norm()) <= 2.5e-3
