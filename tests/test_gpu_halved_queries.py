"""Backward in one launch whose last query blocks are taken in halves (the numbers of blocks at which the rules take some, and
neighbours at which they take none), ragged ends in either half, lists of 0 entries, of one (groups without any), of a few and of
all blocks, the token rule, against float64.  How many each case halves, (caller's lists, token rule), is held against the rules by
tests/test_halved_queries_host.py."""
import pytest

import test_gpu_halved_blocks as halved_blocks
import test_gpu_list_split as list_split

pytestmark = pytest.mark.gpu

CASES = {(3, 43, 100): (64, 64), (5, 34, 1): (128, 128), (10, 17, 64): (128, 128), (8, 50, 127): (64, 64), (9, 34, 63): (128, 128),
         (27, 19, 0): (64, 64), (6, 36, 65): (0, 0)}
CASES_64 = {
    (64, 3, 43 * 64 - 1): (96, 96), (64, 4, 44 * 64): (96, 96), (64, 3, 59 * 64 - 63): (0, 0), (64, 5, 52 * 64 - 31): (192, 192),
    (64, 8, 41 * 64 - 32): (192, 192), (64, 7, 47 * 64): (0, 0), (128, 5, 13 * 128 - 64): (0, 96), (128, 1, 65 * 128 - 64): (96, 96),
    (128, 4, 22 * 128 - 127): (96, 96), (128, 4, 33 * 128 - 1): (192, 192), (128, 4, 41 * 128 - 32): (192, 192),
    (128, 8, 33 * 128 - 65): (192, 192), (128, 8, 41 * 128 - 96): (192, 192), (128, 7, 47 * 128): (0, 0)}


@pytest.mark.parametrize("H, nb, cut", CASES)
@pytest.mark.parametrize("rule", [False, True])
def test_backward_matches_float64(H, nb, cut, rule):
    halved_blocks.test_forward_and_backward_match_float64(128, H, nb, cut, rule)


@pytest.mark.parametrize("block, H, N", CASES_64)
@pytest.mark.parametrize("rule", [False, True])
def test_head_dimension_64_matches_float64(block, H, N, rule):
    list_split.test_forward_and_backward_match_float64(64, block, H, N, rule)
