"""The rule for halves at the end of a common backward launch, as the library compiles it, against the same lists laid out on 256
units one by one, up to the largest common launch."""
import heapq
import os
import shutil
import subprocess

import pytest

from oracle import build as obuild
from paper_2506_19852_amd import build as hip_build
from test_gpu_halved_queries import CASES, CASES_64
from test_launch_form_host import forms  # noqa: F401  (a fixture)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "tests", "host", "halved_queries.hip")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if not os.path.exists(hip_build.HIPCC) and shutil.which(hip_build.HIPCC) is None:
        pytest.skip("hipcc not available")
    exe = tmp_path_factory.mktemp("host") / "halved_queries"
    r = subprocess.run([hip_build.HIPCC, *hip_build.FLAGS, "--cuda-host-only", SOURCE, "-o", str(exe)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]

    def run(cases):
        r = subprocess.run([str(exe)], input="\n".join("%d %d %d" % c for c in cases), stdout=subprocess.PIPE, text=True, timeout=60)
        assert r.returncode == 0
        return [tuple(map(int, line.split())) for line in r.stdout.split("\n") if line]
    return run


def laid_out(items, halved):
    units = [0] * 256
    for n, time in ((items, 40), (items - halved, 31), (2 * halved, 18)):
        for _ in range(n):
            heapq.heapreplace(units, units[0] + time)
    return max(units)


def test_rule_matches_lists_laid_out_one_by_one(rule):
    sizes = sorted({129, 130, 192, 193, 255, 256, 257, 512, 513, 768, 769, 1024, 1535, 1536, *range(128, 1537, 37)})
    for items, got in zip(sizes, rule([(n, 0, 30) for n in sizes])):
        ends = [laid_out(items, h) for h in (0, 64, 128)]
        best = min(ends[1:])
        want = 0 if items <= 128 or 25 * best > 24 * ends[0] else (128 if ends[2] < ends[1] else 64)
        assert got[:4] == (want, *ends), items


def test_no_halves_in_other_launches(rule):
    """Among slices, on lists of a few entries, where every workgroup has a unit, above the sizes of a common launch."""
    assert [r[0] for r in rule([(400, 0, 4), (400, 1, 30), (400, 0, 3), (128, 0, 30), (1, 0, 30), (1537, 0, 30), (100000, 0, 30)])] == [64, 0, 0, 0, 0, 0, 0]


def test_halves_at_head_dimension_64(rule):
    """By dQ's workgroups: 129 to 176, and 1 to 72 above whole rounds of 256; blocks of 128 have two each up to 256 blocks."""
    sizes = [128, 129, 176, 177, 256, 257, 328, 329, 512, 513, 584, 585]
    assert [r[4] for r in rule([(n, 0, 30) for n in sizes])] == [0, 96, 96, 0, 0, 192, 192, 0, 0, 192, 192, 0]
    sizes = [64, 65, 88, 89, 128, 129, 164, 165, 256, 257, 328, 329, 513]
    assert [r[5] for r in rule([(n, 0, 30) for n in sizes])] == [0, 96, 96, 0, 0, 192, 192, 0, 0, 192, 192, 0, 192]
    assert [r[4:] for r in rule([(257, 1, 30), (257, 0, 3), (257, 0, 4)])] == [(0, 0), (0, 0), (192, 192)]


def test_gpu_cases_take_the_halves_they_are_meant_to(forms):  # noqa: F811
    """The launches of tests/test_gpu_halved_queries.py, with the lengths of the lists and the frames that its two tests make."""
    def by_rule(frames, s, block, N):
        bitmap, _ = obuild.mask_scan(frames, s, block, 1, 0, -(-N // block), 1, 1, N - frames * s)
        return int(bitmap.sum()), int(bitmap.sum(1).max())
    launches, want = [], []
    for (H, nb, cut), halved in CASES.items():
        N = 128 * nb - cut
        lists = [nb if r == 3 else (9, 0, 1, 4, 5)[r % 5] for r in range(nb)]
        launches += [(128, 128, H, nb, (sum(lists), max(lists))), (128, 128, H, nb, by_rule(N // 150, 150, 128, N))]
        want += halved
    for (block, H, N), halved in CASES_64.items():
        nb = -(-N // block)
        lists = [(0, 1, 2, 3, 5, nb)[r % 6] for r in range(nb)]
        launches += [(64, block, H, nb, (sum(lists), max(lists))), (64, block, H, nb, by_rule(N // 128, N // (N // 128), block, N))]
        want += halved
    for launch, got, halved in zip(launches, forms(launches, "halves"), want):
        assert got == (halved,), launch
