"""The fp32 configuration's products at the edges of their tiles and K-steps: shares of K of one to 32 values and several steps of
256 (tiles of 32), 256 tiles and more (tiles of 64, K-steps of 32), rows, columns and ranks beside a tile's edge."""
import pytest

from paper_2602_07263_amd import workloads as wk
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

CASES = [
    ("smallest", 8, 8, [1], [1]),
    ("shares_of_four", 16, 24, [1, 3], [1, 2]),
    ("uneven_shares", 136, 40, [5, 33], [31, 34]),
    ("one_step_and_a_rest", 264, 520, [64, 1, 7], [257, 0, 3]),
    ("several_steps", 776, 248, [65, 32], [300, 129]),
    ("tiles_of_64", 1032, 1048, [40, 3], [1030, 27]),
    ("tiles_of_64_whole", 1024, 1024, [64], [1024]),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_f32_products_meet_the_oracle(case):
    name, d_in, d_out, ranks, tokens = case
    p = wk.generate(wk.custom(name, "f32", d_in, d_out, ranks, tokens, [2.0] * len(ranks)), seed=71)
    for reuse in (True, False):
        Y, dX, dA, dB, _ = pu.run_gpu(p, reuse_S=reuse)
        res = pu.compare(p, Y, dX, dA, dB)
        assert all(v <= 1.0 for v in res.values()), f"{name} reuse={reuse}: worst error / tolerance ratios {res}"
