"""Products of an MLP block that share a launch (gate and up, forward and backward) against float64: all tiles cut, a boundary
between the products among whole tiles, ragged widths, a contraction that may not pair, and both sides of the longest pair."""
import pytest

pytestmark = pytest.mark.gpu


def _reference(torch, X, gamma, layers, ranks, off, scales, dOut):
    """Out, dX and {layer: [dA, dB per job]} in float64, by the definition of the block."""
    d = torch.float64
    p = {n: [W.to(d).requires_grad_(False), [a.to(d).requires_grad_() for a in A], [b.to(d).requires_grad_() for b in B]]
         for n, (W, A, B) in layers.items()}
    x = X.to(d).requires_grad_()

    def project(n, h):
        W, A, B = p[n]
        return torch.cat([h[off[j]:off[j + 1]] @ W + scales[j] * (h[off[j]:off[j + 1]] @ A[j]) @ B[j] for j in range(len(ranks))])
    h = x / torch.sqrt((x * x).mean(1, keepdim=True) + 1e-5) * gamma.to(d)
    out = x + project("down", torch.nn.functional.silu(project("gate", h)) * project("up", h))
    out.backward(dOut.to(d))
    return out.detach(), x.grad, {n: [t.grad for t in p[n][1] + p[n][2]] for n in p}


@pytest.mark.parametrize("d,dff,tokens", [(2048, 520, [300, 213]), (2048, 4096, [1500, 600]), (1024, 4104, [2000, 100]),
                                          (64, 4096, [49000, 152]), (64, 4096, [49000, 153])],
                         ids=["all_cut", "boundary_inside", "odd_contraction", "longest_pair", "beyond_it"])
def test_paired_products_match_float64(d, dff, tokens):
    import torch
    from paper_2602_07263_amd import tlora
    g = torch.Generator(device="cuda").manual_seed(d + dff + sum(tokens))
    rnd = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).to(torch.bfloat16)
    ranks, scales, off = [8, 20], [2.0, 0.5], [0, tokens[0], sum(tokens)]
    T = off[-1]
    layers = {n: (rnd(i, o, std=i ** -0.5), [rnd(i, r, std=i ** -0.5) for r in ranks], [rnd(r, o, std=0.05) for r in ranks])
              for n, (i, o) in dict(gate=(d, dff), up=(d, dff), down=(dff, d)).items()}
    X, dOut, gamma = rnd(T, d), rnd(T, d), (1 + 0.1 * torch.randn(d, device="cuda", generator=g)).to(torch.bfloat16)
    blk = tlora.MlpBlock("bf16", d, dff, ranks, off, scales, X, gamma, 1e-5, layers)
    Out, dX = torch.full_like(X, float("nan")), torch.full_like(X, float("nan"))
    grads = blk.new_grads()
    blk.fwd(Out)
    blk.bwd(dOut, dX, grads)
    torch.cuda.synchronize()
    out_r, dx_r, g_r = _reference(torch, X, gamma, layers, ranks, off, scales, dOut)
    # A tensor rounded to bf16 is off by 2^-9 / sqrt(3) = 1.1e-3 of itself in the 2-norm.  At most eight are rounded on the way to
    # any output (normed rows, G, U, Z and its product; dZ, dG, dU and their products behind them): sqrt(8) 1.1e-3 = 3.2e-3 when
    # they add like noise, and twice that is allowed.
    for name, got, want in [("Out", Out, out_r), ("dX", dX, dx_r)] + \
            [(f"{n} {i}", a, b) for n in grads for i, (a, b) in enumerate(zip(grads[n][0] + grads[n][1], g_r[n]))]:
        rel = float((got.double() - want).norm() / want.norm())
        assert rel <= 6.4e-3, (name, rel)
