"""The rules that choose a launch's form, evaluated on the host as the library compiles them: lists too short to
share are not split, whatever the number of items, and the forms change where the rules' comments say."""
import os
import shutil
import subprocess

import pytest

from paper_2506_19852_amd import build as hip_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "tests", "host", "launch_form.hip")


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    if not os.path.exists(hip_build.HIPCC) and shutil.which(hip_build.HIPCC) is None:
        pytest.skip("hipcc not available")
    exe = tmp_path_factory.mktemp("host") / "launch_form"
    r = subprocess.run([hip_build.HIPCC, *hip_build.FLAGS, "--cuda-host-only", SOURCE, "-o", str(exe)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]

    def run(cases, *words):
        """(D, block, heads, n_blocks, entries per list or (total, longest)) -> (forward, dq, dkdv, fp8, heads by length in forward, dq, dkdv)"""
        lines = []
        for D, block, heads, nb, per in cases:
            nnz, longest = (nb * per, per) if isinstance(per, int) else per
            lines.append(f"{D} {block} {heads} {nb} {nnz} {longest} {longest}")
        r = subprocess.run([str(exe), *words], input="\n".join(lines), stdout=subprocess.PIPE, text=True, timeout=60)
        assert r.returncode == 0
        out = [tuple(map(int, line.split())) for line in r.stdout.split("\n") if line]
        assert len(out) == len(cases)
        return out
    return run


def test_short_lists_are_not_split(forms):
    cases = [(D, block, heads, nb, per) for D in (64, 128) for block in (64, 128) for per in (0, 1)
             for heads, nb in ((1, 1), (4, 16), (8, 32), (20, 12), (5, 60), (16, 60), (24, 50), (24, 200), (24, 800))]
    for case, form in zip(cases, forms(cases)):
        assert form[:4] == (1, 1, 1, 1), case
    # two entries pay for half blocks in the backward only (dK/dV and dQ one after the other); three entries for nothing above one round
    assert [f[:4] for f in forms([(128, 128, 4, 16, 2), (128, 128, 4, 16, 3), (128, 128, 8, 32, 3), (64, 64, 16, 60, 3), (64, 64, 24, 200, 6)])] == [
        (1, 4, 2, 1), (4, 4, 2, 1), (1, 1, 1, 1), (1, 1, 1, 1), (1, 1, 1, 1)]


def test_forms_change_at_the_measured_sizes(forms):
    wide = lambda nb: (60 * nb, 120)   # lists of very unequal length
    assert [f[:3] for f in forms([
        # block 128: half blocks to 128 items, two groups to 256
        (128, 128, 8, 16, 16), (128, 128, 3, 43, 16), (128, 128, 8, 32, 16), (128, 128, 1, 257, 16),
        # block 64: four groups to 256 items, two to 512
        (128, 64, 8, 32, 16), (128, 64, 8, 32, 11), (128, 64, 1, 257, 16), (128, 64, 8, 64, 48),
        # to 1024 items: long unequal lists in two groups (dK/dV: 513 to 768 items), or very unequal ones
        (128, 64, 12, 50, 48), (64, 64, 12, 50, (48 * 50, 50)), (64, 64, 12, 50, (23 * 50, 30)), (128, 64, 9, 100, (9600, 109)), (128, 64, 9, 100, 100),
        (128, 64, 9, 100, wide(100)),
        # to 1536: two groups (dK/dV: to 1200); above: D 64 forward, long lists only
        (128, 64, 11, 100, 48), (128, 64, 15, 100, 48), (128, 64, 16, 100, 48), (64, 64, 40, 100, 48), (64, 64, 40, 100, 24)])] == [
        (4, 4, 2), (2, 2, 1), (2, 2, 1), (1, 1, 1),
        (4, 4, 2), (2, 2, 2), (2, 2, 2), (2, 2, 1),
        (1, 1, 2), (2, 2, 2), (1, 1, 1), (2, 2, 1), (1, 1, 1),
        (2, 2, 2),
        (2, 2, 2), (2, 2, 1), (1, 1, 1), (2, 1, 1), (1, 1, 1)]


def test_heads_by_list_length(forms):
    """All heads up to one round of workgroups (256 items; 512 in blocks of 64) and up to 8 heads; else the last ones that
    fit the cache."""
    assert [f[4] for f in forms([(128, 128, 20, 12, 4), (128, 128, 256, 1, 1), (128, 128, 257, 1, 1), (128, 64, 40, 12, 12), (64, 64, 512, 1, 1),
                                 (64, 64, 513, 1, 1), (128, 128, 8, 300, 50), (128, 128, 9, 300, 50), (128, 128, 24, 929, 100),
                                 (128, 128, 1, 16385, 100)])] == [20, 256, 8, 40, 512, 8, 8, 8, 2, 0]


def test_long_heads_in_blocks_of_64_stay_with_slices(forms):
    """On either side of the most K and V per XCD: 28 MiB (forward), 16 MiB (its last 8 of more heads), 64 MiB (dQ).  Blocks
    of 128, dK/dV and launches that last as long as one of their lists have no such limit."""
    skewed = lambda nb: (100 * nb, 200)
    cases = [(128, 64, 4, 896, 100), (128, 64, 4, 897, 100), (64, 64, 4, 1792, 100), (64, 64, 4, 1793, 100), (128, 64, 1, 897, skewed(897)), (128, 64, 4, 1100, skewed(1100)),
             (128, 64, 5, 597, 100), (128, 64, 5, 598, 100), (128, 64, 6, 598, 100), (128, 64, 3, 716, 100), (128, 64, 3, 717, 100),
             (128, 64, 7, 512, 100), (128, 64, 7, 513, 100), (128, 64, 16, 512, 100), (128, 64, 16, 513, 100),
             (128, 64, 2, 2048, 100), (128, 64, 2, 2049, 100), (128, 128, 4, 513, 100), (128, 128, 1, 2056, 100)]
    assert [f[4:] for f in forms(cases)] == [
        (4, 4, 4), (0, 4, 4), (4, 4, 4), (0, 4, 4), (1, 1, 1), (0, 4, 4), (5, 5, 5), (0, 5, 5), (0, 6, 6), (3, 3, 3), (0, 3, 3),
        (7, 7, 7), (0, 7, 7), (8, 8, 8), (0, 8, 8), (0, 2, 2), (0, 0, 2), (4, 4, 4), (1, 1, 1)]


def test_backward_into_the_memory_of_q_or_dout_keeps_its_groups(forms):
    """Such a call runs dK/dV and dQ one after the other, each in the form that is best by itself: small launches are split
    as dense in groups as where dq has memory of its own."""
    after = 0
    cases = [(64, 64, 2, 32, 32), (64, 64, 9, 32, 8), (64, 64, 16, 32, 2), (64, 64, 24, 32, 16), (64, 64, 60, 32, 32), (64, 128, 2, 32, 32), (64, 128, 8, 32, 8),
             (128, 64, 2, 32, 32), (128, 64, 9, 32, 8), (128, 64, 12, 32, 16), (128, 128, 4, 32, 32), (128, 128, 8, 32, 8), (128, 128, 9, 32, 8)]
    assert [f[3:] for f in forms(cases, "backward")] == [
        (after, 2, 4), (after, 2, 2), (after, 1, 1), (after, 1, 1), (after, 2, 1), (after, 2, 4), (after, 1, 2),
        (after, 2, 4), (after, 1, 2), (after, 2, 2), (after, 2, 4), (after, 1, 2), (after, 1, 1)]
    # with memory of its own: one launch in groups (1), by hand (2) or in pairs (3) up to these sizes
    cases = [(64, 64, 2, 32, 1), (64, 64, 2, 33, 1), (64, 64, 48, 32, 4), (64, 64, 49, 32, 4), (64, 128, 1, 32, 1), (64, 128, 8, 32, 1), (64, 128, 8, 33, 1), (64, 128, 48, 33, 1),
             (128, 64, 4, 32, 1), (128, 64, 4, 33, 1), (128, 128, 2, 32, 1), (128, 128, 2, 33, 1), (128, 128, 48, 32, 4), (128, 128, 48, 33, 4)]
    assert [f[:3] for f in forms(cases, "backward")] == [
        (1, 4, 4), (1, 2, 2), (1, 2, 2), (0, 1, 1), (1, 4, 4), (1, 2, 2), (1, 1, 1), (0, 1, 1),
        (2, 2, 2), (0, 1, 1), (2, 2, 2), (3, 1, 2), (3, 1, 2), (0, 1, 1)]


def test_backward_of_very_short_lists_is_one_launch_only_where_that_saves_a_round(forms):
    """D 128 in blocks of 128: lists of one entry up to 384 blocks, of two and three also where the last round of 256 is at most
    half full.  D 64 in blocks of 64: lists of one entry up to 640 blocks."""
    cases = [(128, 128, *c) for c in ((12, 32, 1), (35, 11, 1), (16, 32, 1), (16, 32, 3), (20, 32, 1), (20, 32, 2), (20, 32, 3), (641, 1, 2), (13, 59, 2), (48, 32, 3), (16, 32, 4), (48, 32, 4))]
    assert [f[0] for f in forms(cases, "backward")] == [3, 0, 0, 0, 0, 3, 3, 0, 0, 0, 3, 3]
    assert [f[0] for f in forms([(64, 64, 20, 32, 1), (64, 64, 641, 1, 1), (64, 64, 48, 32, 1), (64, 64, 48, 32, 2), (64, 128, 48, 32, 1)], "backward")] == [1, 0, 0, 1, 1]


def test_forward_forms_ahead_of_the_groups(forms):
    """Groups of one wave while 32-row parts have a compute unit each; halves of the last blocks of 128 up to half a round of 256,
    where all heads go by length; parts of the 8-bit forward to 64 and to 128 blocks.  Lists of one entry in none of them."""
    single = [(64, 64, 4, 32, 2), (128, 64, 129, 1, 2), (64, 64, 4, 32, 1), (128, 128, 2, 32, 2), (64, 128, 65, 1, 2), (128, 128, 2, 32, 1)]
    assert [f[0] for f in forms(single, "forward")] == [1, 0, 0, 1, 0, 0]
    halved = [(128, 128, 8, 32, 16), (128, 128, 1, 257, 16), (128, 128, 12, 32, 16), (64, 128, 5, 77, 16), (128, 128, 16, 32, 16), (128, 128, 20, 32, 4), (128, 128, 20, 32, 3),
              (128, 128, 10, 110, 90), (128, 128, 24, 929, 100)]
    assert [f[1] for f in forms(halved, "forward")] == [0, 1, 128, 0, 0, 128, 0, 76, 0]
    parts = [(128, 128, 2, 32, 2), (128, 128, 5, 13, 2), (128, 128, 4, 32, 2), (128, 128, 3, 43, 2), (128, 128, 2, 32, 1)]
    assert [f[2] for f in forms(parts, "forward")] == [4, 2, 2, 1, 1]


def test_parts_of_blocks_only_where_all_heads_go_by_length(forms):
    """Several workgroups per block are laid over the heads that go by length: every head has to."""
    cases = [(D, block, heads, nb, per) for D in (64, 128) for block in (64, 128) for per in (1, 2, 4, 12, 40)
             for heads, nb in ((1, 1), (1, 64), (1, 128), (3, 43), (16, 8), (64, 2), (65, 2), (128, 1), (128, 2), (9, 28), (20, 12), (256, 1), (300, 1), (17, 33), (2, 900))]
    groups, ahead, back = forms(cases), forms(cases, "forward"), forms(cases, "backward")
    for (D, block, heads, nb, per), g, f, b in zip(cases, groups, ahead, back):
        forward, dq, dkdv = g[4:]
        half = block == 128
        if f[0] or f[1] or f[2] > 1 or (half and g[0] == 4):
            assert forward == heads, (D, block, heads, nb, per)
        # one launch in groups of 32 or 64 rows (D 64), by hand in 64 rows; one after the other in half blocks
        if b[0] == 1 and (b[1] == 4 or (half and b[1] == 2)) or (b[0] == 2 and half):
            assert dq == dkdv == heads, (D, block, heads, nb, per)
        if half and b[4] == 2:
            assert dkdv == heads, (D, block, heads, nb, per)
        if half and b[5] == 4:
            assert dq == heads, (D, block, heads, nb, per)
