"""Shrinks cut into splits whose stages hold 32, 64 or 128 rank columns, on both sides of each width, with fewer K-steps in a split than
stages, as many and more: against the fp64 oracle."""
import pytest

from paper_2602_07263_amd import workloads as wk
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_in,d_out", [(512, 1280), (4096, 704)])
@pytest.mark.parametrize("ranks", [[32, 33], [64, 65], [1, 57]], ids=str)
def test_shrink_stages(d_in, d_out, ranks):
    p = wk.generate(wk.custom("stages", "bf16", d_in, d_out, ranks, [97, 1300], [2.0, 0.5]), seed=17)
    Y, dX, dA, dB, _ = pu.run_gpu(p)
    res = pu.compare(p, Y, dX, dA, dB)
    assert all(v <= 1.0 for v in res.values()), f"worst error / tolerance ratios {res}"
