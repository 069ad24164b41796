"""dK / dV take the two 32-query blocks of a 64-query step on different waves and add their sums: sequences that end in
the first block, at its edge, in the second, and one query past a step, for every key block of a tile."""
import pytest

from tests import test_attention_gpu as ta

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,heads", [([1, 31, 32, 33, 63, 64, 65, 95, 96, 97], (3, 1)),
                                        ([127, 129, 159, 160, 161, 191, 193, 223, 225, 255], (4, 2))],
                         ids=["one_tile", "two_tiles"])
def test_sequences_that_end_in_either_query_block(lens, heads):
    ta.test_attention_fwd_bwd_match_oracle((lens, *heads))
