"""One query head per kv head in 8 bits: scores are joined in registers up to some number of tiles in a launch and go through LDS beyond it. On both
sides of that line, and at its edge, results are those of the plain kernel, with a tail and without; lengths at the edges of tiles."""
import pytest

import paper_2405_12591_amd as dq
from test_gpu_head_sets import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,tiles,registers", [(1, 2, 1), (16, 80, 1), (16, 81, 0), (40, 33, 0)])
@pytest.mark.parametrize("tail", [0, 1])
def test_one_head_in_8_bits_on_both_sides_of_the_line(batch, tiles, registers, tail):
    assert dq.lib.dq_debug_mfma_spread(8 * batch, tiles) == registers
    _compare(8, 128, 1, batch, tiles, tail=tail)
