"""dA / dB whose jobs are one unit (the unit stores the gradient) or several (partial tiles and their sum), in one launch or two:
against the fp64 oracle, overwriting and adding, with ranks that end inside a block of 32 or 128 or off a multiple of 4, idle jobs
and widths off the 256-column tile."""
import pytest

from paper_2602_07263_amd import workloads as wk
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

CASES = [
    ("one_launch_one_unit", 4096, 4160, [16], [200]),
    ("ranks_off_four", 2056, 2112, [1, 3, 30, 130], [31, 65, 1, 129]),
    ("two_blocks_and_idle_jobs", 1032, 3080, [256, 7, 129], [500, 0, 33]),
    ("a_long_job_beside_short_ones", 2048, 2304, [8, 40, 5], [6000, 40, 300]),
    ("long_jobs_of_full_height", 4096, 1024, [128, 64], [4100, 700]),
    ("around_seven_steps", 1024, 1032, [32, 8, 25], [192, 224, 250]),
    ("two_launches", 264, 520, [8, 33, 2], [700, 0, 4500]),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_gradients_meet_the_oracle(case):
    import torch
    from paper_2602_07263_amd import tlora
    name, d_in, d_out, ranks, tokens = case
    p = wk.generate(wk.custom(name, "bf16", d_in, d_out, ranks, tokens, [2.0, 0.5, 1.0, 3.0][:len(ranks)]), seed=81)
    Y, dX, dA, dB, lp = pu.run_gpu(p)
    res = pu.compare(p, Y, dX, dA, dB)
    assert all(v <= 1.0 for v in res.values()), f"{name}: worst error / tolerance ratios {res}"
    # adding: 3 + the gradient, rounded once to fp32
    dY = torch.from_numpy(p.dY).to(device="cuda", dtype=torch.bfloat16)
    _, _, dA2, dB2 = lp.new_outputs()
    for t in dA2 + dB2:
        t.fill_(3.0)
    lp.bwd(dY, None, dA2, dB2, reuse_S=True, flags=tlora.TLORA_BWD_ACCUMULATE)
    torch.cuda.synchronize()
    for got, g in zip(dA2 + dB2, list(dA) + list(dB)):
        want = torch.from_numpy(g).to("cuda") + 3.0
        assert torch.equal(got, want), name


def test_gradients_whose_partial_tiles_have_no_room_together():
    """A long job of the highest rank: dB and dA in a launch each, one after the other through the same room."""
    import torch
    from paper_2602_07263_amd import tlora
    d_in, d_out, r, T, scale = 64, 5120, 1024, 52011, 2.0
    g = torch.Generator(device="cuda").manual_seed(82)
    rnd = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).to(torch.bfloat16)
    X, W, A, B, dY = rnd(T, d_in), rnd(d_in, d_out), rnd(d_in, r, std=d_in ** -0.5), rnd(r, d_out, std=0.01), rnd(T, d_out)
    lp = tlora.LayerProblem("bf16", d_in, d_out, [r], [0, T], [scale], X, W, [A], [B])
    dA, dB = torch.full((d_in, r), 1.0, device="cuda"), torch.full((r, d_out), 1.0, device="cuda")
    for flags, add in ((0, 0.0), (tlora.TLORA_BWD_ACCUMULATE, 1.0)):
        lp.bwd(dY, None, [dA], [dB], flags=flags)
        x, dy, a, b = (t.double() for t in (X, dY, A, B))
        dA_r, dB_r = scale * x.T @ (dy @ b.T), scale * (x @ a).T @ dy
        # S and dS as two bf16 planes: 2^-17 of themselves at most; fp32 sums of at most 4096 tokens, then of 13: 2^-24 sqrt(4096)
        for got, want in ((dA, dA_r), (dB, dB_r)):
            assert float((got.double() - (1.0 + add) * want).norm() / want.norm()) <= 2 * (2.0 ** -17 + 2.0 ** -18), (flags, want.shape)
