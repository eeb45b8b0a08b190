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


def case(n_blocks, sliced, ordered, mean, max_slice=0, codes=0):
    return (n_blocks, sliced, ordered, mean, max_slice or (n_blocks + 7) // 8, codes)


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
