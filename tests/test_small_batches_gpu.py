"""Batches of at most 128 tokens, whose directions run in two launches each (a contraction cut over workgroups and waves, then the
sums, the adapters' second product and the planes): against the fp64 oracle at the edges of their tiles."""
import pytest

from paper_2602_07263_amd import workloads as wk
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

CASES = [
    # name, d_in, d_out, ranks, tokens
    ("one_token", 512, 512, [8], [1]),
    ("a_block_of_16", 576, 640, [3, 40], [15, 1]),                      # 9 and 10 K-steps of 64: a wave with a single step
    ("one_more", 640, 4096, [16, 1, 64], [5, 7, 5]),
    ("half", 4096, 1088, [130, 8], [63, 1]),                            # rank rows beyond two tiles of 64
    ("past_half", 1024, 3008, [8, 256, 5], [1, 63, 1]),
    ("last_but_one", 4096, 4096, [8, 16, 32, 8], [40, 47, 0, 40]),      # an idle job between active ones
    ("all_rows", 2048, 1024, [100, 31, 300], [64, 33, 31]),
    ("no_rank", 512, 1024, [0, 0], [60, 9]),
    ("a_job_without_rank", 832, 512, [0, 24, 0], [3, 50, 20]),
    ("one_rank_each", 512, 576, [1] * 128, [1] * 128),
    ("largest_rank", 512, 512, [1024], [17]),
    ("more_idle_rank_rows_than_active", 512, 512, [8, 64, 64], [9, 0, 0]),      # keeps the general kernels
    ("one_token_too_many", 512, 512, [8, 5], [100, 29]),                        # so does this
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_small_batches_meet_the_oracle(case):
    from paper_2602_07263_amd import tlora
    name, d_in, d_out, ranks, tokens = case
    p = wk.generate(wk.custom(name, "bf16", d_in, d_out, ranks, tokens, [2.0] * len(ranks)), seed=61)
    cuts = tlora.tlora_plan_cuts(tlora.LayerProblem.from_numpy(p).prob)
    small = name not in ("more_idle_rank_rows_than_active", "one_token_too_many")
    assert (cuts["fwd"] == (0, cuts["shrink_x"]) and cuts["bwd"] == (0, cuts["shrink_dy"])) == small, cuts
    for reuse in (True, False):
        Y, dX, dA, dB, _ = pu.run_gpu(p, reuse_S=reuse)
        res = pu.compare(p, Y, dX, dA, dB)
        assert all(v <= 1.0 for v in res.values()), f"{name} reuse={reuse}: worst error / tolerance ratios {res}"


# The backward of dY is small while the forward is not, so a backward that makes S again runs both forms in one room of sums:
# dY's fragments (33 tokens on) lie behind whichever sums are more.
HALF_SMALL = [
    # name, d_in, d_out, ranks, tokens
    ("twelve_short_jobs", 12288, 4096, [128] * 12, [3] * 12),
    ("three_jobs", 5248, 512, [768, 128, 512], [28, 33, 24]),
    ("four_jobs_110_tokens", 4672, 576, [256, 1024, 512, 64], [27, 28, 27, 28]),
]


@pytest.mark.parametrize("case", HALF_SMALL, ids=[c[0] for c in HALF_SMALL])
def test_small_backward_of_a_general_forward(case):
    from paper_2602_07263_amd import tlora
    name, d_in, d_out, ranks, tokens = case
    p = wk.generate(wk.custom(name, "bf16", d_in, d_out, ranks, tokens, [2.0] * len(ranks)), seed=63)
    cuts = tlora.tlora_plan_cuts(tlora.LayerProblem.from_numpy(p).prob)
    assert cuts["fwd"] != (0, cuts["shrink_x"]) and cuts["bwd"] == (0, cuts["shrink_dy"]), cuts
    for reuse in (True, False):
        Y, dX, dA, dB, _ = pu.run_gpu(p, reuse_S=reuse)
        res = pu.compare(p, Y, dX, dA, dB)
        assert all(v <= 1.0 for v in res.values()), f"{name} reuse={reuse}: worst error / tolerance ratios {res}"


def test_row_lists_scratch_and_partial_outputs_give_the_same_bits():
    """Through a row list, without an allocation, without dX and without gradients: the plain call's bits."""
    import torch
    from paper_2602_07263_amd import tlora
    d_in, d_out, ranks, tokens = 1024, 640, [8, 40], [70, 31]
    p = wk.generate(wk.custom("small", "bf16", d_in, d_out, ranks, tokens, [2.0, 1.0]), seed=62)
    lp = tlora.LayerProblem.from_numpy(p)
    dY = torch.from_numpy(p.dY).to(device="cuda", dtype=torch.bfloat16)
    Y, dX, dA, dB = lp.new_outputs()
    lp.fwd(Y)
    lp.bwd(dY, dX, dA, dB, reuse_S=True)
    index = torch.randperm(101, generator=torch.Generator().manual_seed(1)).to(torch.int32).cuda()
    at = index.long()
    X2, dY2 = torch.empty_like(lp.X), torch.empty_like(dY)
    X2[at], dY2[at] = lp.X, dY
    lq = tlora.LayerProblem("bf16", d_in, d_out, ranks, p.offsets, [2.0, 1.0], X2, lp.W, lp.A, lp.B)
    Y2, dX2, dA2, dB2 = lq.new_outputs()
    n = tlora.tlora_indexed_workspace_bytes(lq.prob)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    st = int(torch.cuda.current_stream().cuda_stream)
    tlora.tlora_fwd_indexed(lq.prob, index.data_ptr(), Y2.data_ptr(), ws.data_ptr(), n, st)
    tlora.tlora_bwd_indexed(lq.prob, index.data_ptr(), dY2.data_ptr(), dX2.data_ptr(), [t.data_ptr() for t in dA2],
                            [t.data_ptr() for t in dB2], tlora.TLORA_BWD_REUSE_S, ws.data_ptr(), n, st)
    Y3, dX3, dA3, dB3 = lp.new_outputs()
    tlora.tlora_fwd_noalloc(lp.prob, Y3.data_ptr(), st)
    lp.fwd(Y)
    lp.bwd(dY, None, dA3, dB3, reuse_S=True)
    lp.bwd(dY, dX3, None, None)
    torch.cuda.synchronize()
    assert torch.equal(Y2[at], Y) and torch.equal(dX2[at], dX) and torch.equal(Y3, Y) and torch.equal(dX3, dX)
    for other in (dA2 + dB2, dA3 + dB3):
        assert all(torch.equal(a, b) for a, b in zip(other, dA + dB))
