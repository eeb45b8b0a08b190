"""Backward of head dimension 128 in blocks of 128 whose last query blocks are taken in halves (the numbers of blocks at which the rule
takes 64 and 128 of them, and neighbours at which it takes none), ragged ends in either half, lists of 0 entries, of one (groups
without any), of a few and of all blocks, the token rule, against float64."""
import pytest

import test_gpu_halved_blocks as halved_blocks

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H, nb, cut", [(3, 43, 100), (5, 34, 1), (10, 17, 64), (8, 50, 127), (9, 34, 63), (27, 19, 0), (6, 36, 65)])
@pytest.mark.parametrize("rule", [False, True])
def test_backward_matches_float64(H, nb, cut, rule):
    halved_blocks.test_forward_and_backward_match_float64(128, H, nb, cut, rule)
