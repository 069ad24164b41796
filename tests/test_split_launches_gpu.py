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
    ("no_rank_at_all", 1024, 2048, [0, 0], [40, 300]),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_split_launches_meet_the_oracle(case):
    name, d_in, d_out, ranks, tokens = case
    p = wk.generate(wk.custom(name, "bf16", d_in, d_out, ranks, tokens, [2.0] * len(ranks)), seed=51)
    for reuse in (True, False):
        Y, dX, dA, dB, _ = pu.run_gpu(p, reuse_S=reuse)
        res = pu.compare(p, Y, dX, dA, dB)
        assert all(v <= 1.0 for v in res.values()), f"{name} reuse={reuse}: worst error / tolerance ratios {res}"
