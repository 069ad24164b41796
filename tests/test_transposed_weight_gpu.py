"""dX of a small batch runs against W as it lies, of a large one against a transposed copy of W: the same bits, and
TLORA_BWD_REUSE_WT finds a copy of the right W whatever the calls before it did."""
import numpy as np
import pytest

from paper_2602_07263_amd import workloads as wk
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

D_IN, D_OUT = 1032, 520          # just above 2^19 elements; K-steps of 32 with a remainder in both directions


def _layer(d_in, d_out, tokens, seed):
    import torch
    from paper_2602_07263_amd import tlora
    p = wk.generate(wk.custom("wt", "bf16", d_in, d_out, [8, 24], tokens, [2.0, 0.5]), seed=seed)
    lp = tlora.LayerProblem.from_numpy(p)
    return p, lp, torch.from_numpy(p.dY).to(device="cuda", dtype=torch.bfloat16)


def _backward(lp, dY, flags=0, forward=True):
    import torch
    Y, dX, dA, dB = lp.new_outputs()
    for t in (Y, dX, *dA, *dB):
        t.fill_(float("nan"))
    if forward:
        lp.fwd(Y)
    lp.bwd(dY, dX, dA, dB, reuse_S=forward, flags=flags)
    torch.cuda.synchronize()
    return [Y, dX, *dA, *dB]


def _same(a, b):
    import torch
    return all(torch.equal(x, y) for x, y in zip(a, b))


# 6144 tokens is the last batch without a copy; K % 32 != 0, = 0 with cut tiles, one token
@pytest.mark.parametrize("d_in,d_out,tokens", [(D_IN, D_OUT, [300, 33]), (1024, 544, [6000, 144]), (1024, 544, [6000, 145]),
                                               (4096, 1024, [1, 0]), (1024, 2048, [700, 500])],
                         ids=["k_tail", "last_without", "first_with", "one_token", "cut"])
def test_with_and_without_the_copy_give_the_same_bits(d_in, d_out, tokens):
    from paper_2602_07263_amd import tlora
    p, lp, dY = _layer(d_in, d_out, tokens, 5)
    try:
        tlora.tlora_set_option("dx_transposed_w", 0)
        lies = _backward(lp, dY)
    finally:
        tlora.tlora_set_option("dx_transposed_w", 1)
    default, redone = _backward(lp, dY), _backward(lp, dY, forward=False)
    assert _same(lies, default) and _same(lies[1:], redone[1:])
    assert _same(lies, _backward(lp, dY, tlora.TLORA_BWD_REUSE_WT)), "the flag after calls without a copy"
    assert _same(lies, _backward(lp, dY, tlora.TLORA_BWD_REUSE_WT)), "and again, now that there is one"
    Y, dX, dA, dB = (default[0], default[1], default[2:4], default[4:6])
    n = lambda t: t.float().cpu().numpy()
    rows = pu.sample_rows(p.offsets, 64, np.random.default_rng(1), per_job=64)
    res = pu.compare(p, n(Y), n(dX), [n(a) for a in dA], [n(b) for b in dB], rows=rows)
    assert all(v <= 1.0 for v in res.values()), res


def test_a_copy_of_another_weight_is_not_taken_for_this_one():
    """Large batch with W (copy), W replaced, small batch (no copy), then the flag: the copy must be of the new W."""
    from paper_2602_07263_amd import tlora
    _, large, dYl = _layer(1024, 544, [6000, 500], 6)
    _, small, dYs = _layer(1024, 544, [200, 100], 7)
    small = tlora.LayerProblem("bf16", 1024, 544, [8, 24], small.offsets, [2.0, 0.5], small.X, large.W, small.A, small.B)
    small.ws, small.ws_bytes = large.ws, large.ws_bytes
    _backward(large, dYl)
    large.W.mul_(-0.5)
    ref = _backward(small, dYs)
    assert _same(ref, _backward(small, dYs, tlora.TLORA_BWD_REUSE_WT))
    ref = _backward(large, dYl)
    assert _same(ref, _backward(large, dYl, tlora.TLORA_BWD_REUSE_WT))


@pytest.mark.parametrize("tokens", [[4096, 2560], [1024, 512]], ids=["with_a_copy", "without"])
def test_nano_batches_share_the_copy_or_do_without(tokens):
    import torch
    from paper_2602_07263_amd import tlora
    p, lp, dY = _layer(1024, 544, tokens, 8)
    ref = _backward(lp, dY)
    for n in (1, 3):
        outs = lp.new_outputs()
        for flags in (0, tlora.TLORA_BWD_REUSE_WT):
            Y, dX, dA, dB = outs
            for t in (Y, dX, *dA, *dB):
                t.fill_(float("nan"))
            lp.fwd_nano(n, 128, Y)
            lp.bwd_nano(n, 128, dY, dX, dA, dB, flags=flags)
            torch.cuda.synchronize()
            # n = 1 is the plain call; smaller batches may cut their sums otherwise: a unit in the last place of bf16
            a, b = dX.float(), ref[1].float()
            assert torch.equal(a, b) if n == 1 else bool(((a - b).abs() <= 2.0 ** -7 * torch.maximum(a.abs(), b.abs()) + 1e-4).all())
