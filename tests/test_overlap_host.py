"""Which tensors of a backward call may share memory, evaluated on the host as the library compiles it: slices of one buffer that
have no element in common do not, and whatever has one does."""
import itertools
import os
import random
import shutil
import subprocess

import pytest

from paper_2506_19852_amd import build as hip_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def may_overlap(tmp_path_factory):
    if not os.path.exists(hip_build.HIPCC) and shutil.which(hip_build.HIPCC) is None:
        pytest.skip("hipcc not available")
    exe = tmp_path_factory.mktemp("host") / "overlap"
    r = subprocess.run([hip_build.HIPCC, *hip_build.FLAGS, "--cuda-host-only", os.path.join(ROOT, "tests", "host", "overlap.hip"), "-o", str(exe)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]

    def run(cases):
        """(B, H, N, D, offset, strides of the first, strides of the second) -> bool"""
        lines = [" ".join(map(str, (*c[:5], *c[5], *c[6]))) for c in cases]
        r = subprocess.run([str(exe)], input="\n".join(lines), stdout=subprocess.PIPE, text=True, timeout=60)
        assert r.returncode == 0
        out = [line == "1" for line in r.stdout.split()]
        assert len(out) == len(cases)
        return out
    return run


def test_slices_of_one_buffer_are_apart(may_overlap):
    cases = []
    for B, H, N, D in ((1, 1, 100, 64), (1, 5, 333, 128), (2, 4, 1000, 64), (3, 2, 1, 128), (2, 1, 7, 128)):
        packed = (N * 4 * H * D, D, 4 * H * D)        # [B, N, 4, H, D]
        side_by_side = (H * N * 2 * D, N * 2 * D, 2 * D)  # [B, H, N, 2, D]
        heads = (N * 2 * H * D, D, 2 * H * D)         # [B, N, 2 H, D]
        stacked = (4 * H * N * D, N * D, D)           # [B, 4, H, N, D]
        for k in (1, 2, 3, -1, -3):
            cases += [(B, H, N, D, k * H * D, packed, packed), (B, H, N, D, k * H * N * D, stacked, stacked)]
        for k in (1, -1):
            cases += [(B, H, N, D, k * D, side_by_side, side_by_side), (B, H, N, D, k * H * D, heads, heads)]
    assert may_overlap(cases) == [False] * len(cases)
    # the first 2 of 4 slices seen as one tensor of twice the heads, and the third
    assert may_overlap([(1, 8, 50, 64, 0, (0, 64, 16 * 64), (0, 64, 16 * 64)), (1, 8, 50, 64, 4 * 64, (0, 64, 16 * 64), (0, 64, 16 * 64)),
                        (1, 8, 50, 64, 8 * 64, (0, 64, 16 * 64), (0, 64, 16 * 64))]) == [True, True, False]


def test_shared_elements_are_never_missed(may_overlap):
    rng = random.Random(5)
    cases, shared = [], []
    for _ in range(4000):
        B, H, N, D = rng.choice((1, 2, 3)), rng.choice((1, 2, 3)), rng.choice((1, 2, 4, 5)), 8
        pick = lambda: (8 * rng.randint(0, 40), 8 * rng.randint(0, 20), 8 * rng.randint(1, 12))
        x = pick()
        y = x if rng.random() < 0.7 else pick()
        offset = 8 * rng.randint(-60, 60)
        rows = lambda s: {b * s[0] + h * s[1] + n * s[2] for b, h, n in itertools.product(range(B), range(H), range(N))}
        cases.append((B, H, N, D, offset, x, y))
        shared.append(not rows(x).isdisjoint({offset + r for r in rows(y)}))   # rows start at multiples of 8 = D
    got = may_overlap(cases)
    assert all(g for g, s in zip(got, shared) if s)
    assert sum(shared) > 500 and sum(not g for g in got) > 500
