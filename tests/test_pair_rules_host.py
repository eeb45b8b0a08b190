"""Which launches go over pairs of neighbouring blocks, at the edges of the rules."""
import os
import shutil
import subprocess

import pytest

from paper_2506_19852_amd import build as hip_build

SOURCE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host", "pair_rules.hip")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if not os.path.exists(hip_build.HIPCC) and shutil.which(hip_build.HIPCC) is None:
        pytest.skip("hipcc not available")
    exe = tmp_path_factory.mktemp("host") / "pair_rules"
    r = subprocess.run([hip_build.HIPCC, *hip_build.FLAGS, "--cuda-host-only", SOURCE, "-o", str(exe)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]

    def run(cases):
        r = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), stdout=subprocess.PIPE, text=True, timeout=60)
        assert r.returncode == 0
        return [int(x) for x in r.stdout.split()]
    return run


def case(n_blocks, sliced, ordered, mean, max_slice=0, codes=0, longest=0, shorter=0, alike=1):
    return (n_blocks, sliced, ordered, mean, max_slice or (n_blocks + 7) // 8, codes, longest or mean, (longest or mean) + (shorter or mean), alike)


def test_fewer_than_8_blocks(rules):
    """One and two blocks always; four from 256 pairs, five and six from 600; three and seven never (an odd last block is a pair of its own)."""
    heads = {1: (280, 5000), 2: (130, 1000), 3: (96, 400, 1000), 4: (65, 80, 127, 128, 600), 5: (53, 120, 199, 200, 400), 6: (48, 64, 199, 200, 400), 7: (40, 80, 160, 700)}
    got = {nb: rules([case(nb, h - 8, 8, nb) for h in hs]) for nb, hs in heads.items()}
    assert got == {1: [1, 1], 2: [1, 1], 3: [0, 0, 0], 4: [0, 0, 0, 1, 1], 5: [0, 0, 0, 1, 1], 6: [0, 0, 0, 1, 1], 7: [0, 0, 0, 0]}
    # 8-bit scores alike
    assert rules([case(3, 88, 8, 3, codes=1), case(4, 57, 8, 4, codes=1), case(4, 120, 8, 4, codes=1)]) == [0, 0, 1]


def test_short_lists_by_slices(rules):
    """From 28 entries on, or where slices start an eighth more workgroups than there are blocks; with 8-bit scores always."""
    assert rules([case(128, 32, 8, m) for m in (1, 2, 10, 27, 28, 128)]) == [0, 0, 0, 0, 1, 1]
    assert rules([case(128, 32, 8, m, codes=1) for m in (1, 2, 27)]) == [1, 1, 1]
    # 8 workgroups for the longest slice: 72 for 64 blocks are an eighth more, for 65 (66 with the last pair's) not; equal slices otherwise
    assert rules([case(64, 40, 8, 5, s) for s in (8, 9)] + [case(65, 40, 8, 5, 9)]) == [0, 1, 0]
    assert rules([case(nb, 200, 8, 2) for nb in (8, 9, 11, 14, 15, 16, 17, 20, 22, 24, 25)]) == [0, 1, 1, 1, 0, 0, 1, 1, 0, 0, 1]


def test_by_length(rules):
    """A whole round of pairs, lists of 64."""
    assert rules([case(110, 0, 10, 93), case(110, 0, 9, 93), case(110, 0, 10, 63), case(16384, 0, 1, 64), case(16385, 0, 1, 64)]) == [1, 0, 0, 1, 0]


def test_lists_with_little_in_common(rules):
    """Only where slices start half as many workgroups again as there are blocks, or heads have fewer than 8 blocks."""
    cases = [(110, 0, 10, 93), (128, 32, 8, 40), (9, 282, 8, 2), (2, 132, 8, 1)]
    assert [rules([case(*c, codes=codes, alike=0) for c in cases]) for codes in (0, 1)] == [[0, 0, 1, 1]] * 2
    assert rules([case(*c) for c in cases]) == [1, 1, 1, 1]
    assert rules([case(128, 32, 8, 5, s, alike=0) for s in (23, 24)]) == [0, 1]


def test_two_long_neighbours(rules):
    """Not where the shorter list of the longest pair (beside slices: at least twice the mean) is more than a workgroup of a whole round has: by length 0.8 of it, 0.95 with 8-bit scores; the last
    heads by length all of it; a fifth where all heads go by slices, 8-bit scores whatever it is."""
    def at(nb, sliced, ordered, mean, share, codes=0):
        shorter = int(share * (ordered or sliced) * nb * mean / 512)
        return case(nb, sliced, ordered, mean, 0, codes, max(nb, shorter), shorter)
    assert rules([at(1971, 0, 1, 606, x) for x in (0.5, 0.79, 0.81, 1.1)]) == [1, 1, 0, 0]
    assert rules([at(1971, 0, 1, 606, x, 1) for x in (0.81, 0.94, 0.96)]) == [1, 1, 0]
    assert rules([at(1804, 3, 1, 582, x) for x in (0.88, 0.99, 1.01)]) == [1, 1, 0]
    assert rules([at(128, 32, 8, 33, x) for x in (0.99, 1.9)] + [at(128, 32, 8, 33, x, 1) for x in (0.94, 1.9)]) == [1, 0, 1, 0]
    assert rules([at(3633, 4, 0, 819, x) for x in (0.16, 0.19, 0.21)] + [at(3633, 2, 0, 819, 0.31, 1)]) == [1, 1, 0, 1]
    assert rules([case(531, 0, 2, 269, longest=531, shorter=531), case(361, 0, 3, 200, longest=361, shorter=361)]) == [0, 0]    # less than twice the mean
    # neighbours that are not twice as long as the others, however short the launch; one long list beside a usual one
    assert rules([case(128, 32, 8, 33, longest=128, shorter=x) for x in (33, 65, 67, 128)] + [case(9, 282, 8, 2)]) == [1, 1, 0, 0, 1]
    # one long list beside usual ones: more than 1.5 of a workgroup's share by length, 3 for the last heads by length; not with 8-bit scores
    assert rules([case(929, 0, 4, 66, longest=x) for x in (718, 719)] + [case(929, 0, 4, 66, codes=1, longest=929)]) == [1, 0, 1]
    assert rules([case(929, 6, 2, 66, longest=x) for x in (718, 719)] + [case(929, 6, 0, 66, longest=929)]) == [1, 0, 1]
    # fewer than 8 blocks: one list can be no longer than the others by much
    assert rules([case(2, 132, 8, 1, longest=2, shorter=2), case(4, 120, 8, 1, longest=4, shorter=4)]) == [1, 1]


def test_key_blocks(rules):
    """Above 1536 blocks: lists of 7 entries, fewer than 8 blocks but for 3 and 7, slices that leave gaps."""
    def keys(*c, s=0):
        return case(*c, s, 2)
    assert rules([keys(128, 4, 8, 7), keys(128, 5, 8, 6), keys(128, 5, 8, 7), keys(129, 0, 12, 7), keys(16384, 1, 0, 7), keys(16385, 1, 0, 7)]) == [0, 0, 1, 1, 1, 0]
    assert rules([keys(nb, 1600, 8, 1) for nb in range(1, 8)] + [keys(7, 400, 8, 7)]) == [1, 1, 0, 1, 1, 1, 0, 1]
    assert rules([keys(nb, 300, 8, 2) for nb in (8, 9, 14, 15, 16, 17)] + [keys(9, 0, 175, 2)]) == [0, 1, 1, 0, 0, 1, 0]
