"""Launches whose contraction is cut into splits because the problem has too few tiles to fill the chip: against the
fp64 oracle, at the sizes where the cut can go wrong -- the fewest K-steps that are split, step counts that the splits do
not divide, one token, jobs without tokens or rank inside a row tile, ranks beyond one column block, ragged row tiles."""
import pytest

from paper_2602_07263_amd import workloads as wk
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

CASES = [
    # name, d_in, d_out, ranks, tokens
    ("fewest_steps", 512, 576, [8, 16], [5, 300]),                       # 8 and 9 K-steps of 64: two splits, 4 + 4 and 4 + 5
    ("one_token", 4096, 1024, [1], [1]),                                 # 16 splits of 4 steps, four of 4
    ("tiny_jobs_in_a_tile", 2048, 640, [3, 0, 40, 8, 130, 7], [1, 4, 31, 0, 33, 16]),
    ("two_column_blocks", 832, 1216, [256, 129, 5], [64, 255, 3]),       # 13 and 19 K-steps
    ("ragged_row_tiles", 1088, 4160, [16, 4, 100], [257, 511, 1]),
    ("many_jobs_in_a_tile", 512, 512, [2, 5] * 150, [1, 0] * 149 + [20, 9]),   # 300 jobs within one row tile
    # a row's job is found among all those of its tile: 257 with one idle, and thousands of idle ones between two active
    ("one_idle_of_257", 512, 512, [1] * 257, [1] * 100 + [0] + [1] * 155 + [2]),
    ("idle_jobs_between_active", 512, 512, [8] * 2500, [5] + [0] * 2498 + [7]),
    ("no_rank_at_all", 1024, 2048, [0, 0], [40, 300]),
    # backbone GEMM: 288 tiles forward, of which the last 32 are cut (65 to 69 steps); 72 of 257 backward, all cut
    ("cut_tiles_after_whole_ones", 2048, 8192, [8, 64, 16], [1000, 3, 1100]),
    ("one_step_too_many", 2080, 264, [8], [255]),                        # 66 steps: eleven shares of 6, ragged columns
    ("short_tile_beside_a_long_one", 512, 512, [8] * 251, [1] * 250 + [40]),   # 79 and 17 steps in seven shares: two are empty
    ("k_tail_is_not_cut", 2056, 512, [8, 5], [100, 29]),
]

CUT_INDEXED = (2048, 1024, [8, 40], [700, 301])


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_split_launches_meet_the_oracle(case):
    name, d_in, d_out, ranks, tokens = case
    p = wk.generate(wk.custom(name, "bf16", d_in, d_out, ranks, tokens, [2.0] * len(ranks)), seed=51)
    for reuse in (True, False):
        Y, dX, dA, dB, _ = pu.run_gpu(p, reuse_S=reuse)
        res = pu.compare(p, Y, dX, dA, dB)
        assert all(v <= 1.0 for v in res.values()), f"{name} reuse={reuse}: worst error / tolerance ratios {res}"


def test_row_list_calls_are_cut_like_the_plain_ones():
    """Same plan, rows fetched and stored through a list: the same bits as the plain call on the sorted rows."""
    import torch
    from paper_2602_07263_amd import tlora
    p = wk.generate(wk.custom("cut_indexed", "bf16", *CUT_INDEXED, [2.0, 1.0]), seed=52)
    lp = tlora.LayerProblem.from_numpy(p)
    T = lp.X.shape[0]
    dY = torch.from_numpy(p.dY).to(device="cuda", dtype=torch.bfloat16)
    Y, dX, dA, dB = lp.new_outputs()
    lp.fwd(Y)
    lp.bwd(dY, dX, dA, dB, reuse_S=True)
    index = torch.randperm(T, generator=torch.Generator().manual_seed(1)).to(torch.int32).cuda()
    at = index.long()
    X2, dY2 = torch.empty_like(lp.X), torch.empty_like(dY)
    X2[at], dY2[at] = lp.X, dY
    lq = tlora.LayerProblem("bf16", 2048, 1024, [8, 40], p.offsets, [2.0, 1.0], X2, lp.W, lp.A, lp.B)
    Y2, dX2, dA2, dB2 = lq.new_outputs()
    n = tlora.tlora_indexed_workspace_bytes(lq.prob)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    st = int(torch.cuda.current_stream().cuda_stream)
    tlora.tlora_fwd_indexed(lq.prob, index.data_ptr(), Y2.data_ptr(), ws.data_ptr(), n, st)
    tlora.tlora_bwd_indexed(lq.prob, index.data_ptr(), dY2.data_ptr(), dX2.data_ptr(), [t.data_ptr() for t in dA2],
                            [t.data_ptr() for t in dB2], tlora.TLORA_BWD_REUSE_S, ws.data_ptr(), n, st)
    torch.cuda.synchronize()
    assert torch.equal(Y2[at], Y) and torch.equal(dX2[at], dX)
    assert all(torch.equal(a, b) for a, b in zip(dA2 + dB2, dA + dB))


def test_a_job_that_is_cut_otherwise_alone_agrees_to_a_rounding():
    """Whether and how a contraction is cut follows from the whole call's shape, so a job's rows may differ between a fused call
    and one of its own by the order of fp32 sums: one unit in the last place of a bf16 value, or, where terms cancel, the
    error of a sum of 2048 products of size |x w| ~ 0.013 (worst order 2048^2 2^-24 0.013 = 3e-3, typically 1e-5)."""
    import torch
    from paper_2602_07263_amd import tlora
    p = wk.generate(wk.custom("fused", "bf16", 2048, 2048, [8, 40, 16], [300, 700, 1900], [2.0, 1.0, 0.5]), seed=53)
    lp = tlora.LayerProblem.from_numpy(p)
    dY = torch.from_numpy(p.dY).to(device="cuda", dtype=torch.bfloat16)
    Y, dX, dA, dB = lp.new_outputs()
    lp.fwd(Y)
    lp.bwd(dY, dX, dA, dB, reuse_S=True)
    fused = tlora.tlora_plan_cuts(lp.prob)
    for j in range(2):
        lo, hi = lp.offsets[j], lp.offsets[j + 1]
        one = lp.job_slice(j)
        alone = tlora.tlora_plan_cuts(one.prob)
        assert alone["fwd"][1] > 1 and alone["fwd"] != fused["fwd"] and alone["shrink_x"] != fused["shrink_x"]
        Y1, dX1, dA1, dB1 = one.new_outputs()
        one.fwd(Y1)
        one.bwd(dY[lo:hi], dX1, dA1, dB1, reuse_S=True)
        torch.cuda.synchronize()
        for a, b in ((Y1, Y[lo:hi]), (dX1, dX[lo:hi])):
            a, b = a.float(), b.float()
            assert bool(((a - b).abs() <= 2.0 ** -7 * torch.maximum(a.abs(), b.abs()) + 1e-4).all())
            assert float((a != b).float().mean()) < 0.02                 # few sums lie that close to a rounding edge
        for a, b in zip(dA1 + dB1, [dA[j], dB[j]]):
            assert bool(((a - b).abs() <= 1e-4 * (1.0 + b.abs())).all())
