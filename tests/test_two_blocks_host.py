"""Every block is taken once by a launch over pairs of query (or key) blocks: whole pairs, single blocks and halves of blocks, by slices and
by length, for even and odd numbers of blocks and slices of any length, and every block has a trace record of its own."""
import os
import random
import shutil
import subprocess

import pytest

from paper_2506_19852_amd import build as hip_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "tests", "host", "two_blocks.hip")


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    if not os.path.exists(hip_build.HIPCC) and shutil.which(hip_build.HIPCC) is None:
        pytest.skip("hipcc not available")
    exe = tmp_path_factory.mktemp("host") / "two_blocks"
    r = subprocess.run([hip_build.HIPCC, *hip_build.FLAGS, "--cuda-host-only", SOURCE, "-o", str(exe)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]

    def run(cases):
        text = "\n".join(" ".join(map(str, (*c[:4], c[5] if len(c) > 5 else 0, *c[4]))) for c in cases)
        r = subprocess.run([str(exe)], input=text, stdout=subprocess.PIPE, text=True, timeout=120)
        assert r.returncode == 0
        parts = [p.strip().split("\n") for p in r.stdout.split("end\n") if p.strip()]
        return [(tuple(map(int, p[0].split())), [tuple(map(int, line.split())) for line in p[1:]]) for p in parts]
    return run


def even_slices(nb):
    return [nb * k // 8 for k in range(9)]


def uneven_slices(nb, seed):
    rng = random.Random(seed)
    return [0, *sorted(rng.randint(0, nb) for _ in range(7)), nb]


CASES = [(nb, sliced, ordered, 100, slices(nb), *codes) for codes in ((), (1,), (2,)) for nb in (1, 2, 3, 7, 8, 9, 15, 16, 17, 64, 101, 110, 929)
         for sliced, ordered in ((0, 10), (1, 8), (8, 0), (9, 8), (17, 2), (32, 8))
         for slices in (even_slices, lambda n: uneven_slices(n, 3 * n + 1))]


def test_every_block_is_taken_once(launches):
    for case, ((_, _, records), items) in zip(CASES, launches(CASES)):
        nb, sliced, ordered = case[:3]
        taken = {}
        for bh, block, half, form, *_ in items:
            for part in [(bh, block, h) for h in (0, 1)] + [(bh, block + 1, h) for h in (0, 1)] if form == 0 else [(bh, block, 0), (bh, block, 1)] if form == 1 else [(bh, block, half)]:
                assert part not in taken, (case, part)
                taken[part] = form
        want = {(bh, block, half) for bh in range(sliced + ordered) for block in range(nb) for half in (0, 1)}
        assert want <= set(taken), (case, sorted(want - set(taken))[:5])
        assert all(block == nb and nb % 2 for _, block, _ in set(taken) - want), case    # the block after an odd last one is in no list
        if len(case) > 5:     # only the bf16 forward is traced
            continue
        written = [r for _, block, half, form, record, _ in items if half == 0 for r in ([record, record + 8] if form == 0 and block + 1 < nb else [record])]
        assert len(written) == len(set(written)) == (sliced + ordered) * nb and min(written) >= 0 and max(written) < records, case
        same = [record % 8 == workgroup % 8 for _, _, _, form, record, workgroup in items if form != 2]
        assert all(same), case


def test_rule(launches):
    """By slices from lists of 28 blocks on; by length from a round of pairs and lists of 64 on; not without the order of the pairs."""
    cases = [(110, 0, 10, 93, even_slices(110)), (110, 0, 9, 93, even_slices(110)), (110, 0, 10, 63, even_slices(110)), (110, 1, 8, 28, even_slices(110)),
             (16384, 1, 0, 28, even_slices(16384)), (16385, 1, 0, 28, even_slices(16385))]
    assert [head[0] for head, _ in launches(cases)] == [1, 0, 0, 1, 1, 0]


def test_whole_rounds_of_pairs_and_halves_at_the_end(launches):
    forms = []
    for _, items in launches([(110, 0, 10, 93, even_slices(110)), (930, 0, 3, 347, even_slices(930)), (256, 32, 8, 160, even_slices(256)), (930, 22, 2, 400, even_slices(930))]):
        forms.append([sum(1 for i in items if i[3] == form) for form in (0, 1, 2)])
    assert forms == [[512, 0, 4 * 38], [1024, 2 * (371 - 64), 4 * 64], [32 * 128 + 512, 2 * (512 - 64), 4 * 64], [22 * 465 + 512, 2 * (418 - 64), 4 * 64]]


def test_single_blocks_with_8_bit_scores(launches):
    """Left over above whole rounds of 512 pairs, in order of length: all up to 192 pairs, none to 256, what is above 256 (at least 64) to 384, none."""
    pairs = {512: 0, 513: 1, 704: 192, 705: 0, 768: 0, 769: 64, 831: 64, 832: 64, 833: 65, 896: 128, 897: 0, 1023: 0, 1024: 0}
    singles = [sum(1 for i in items if i[3] == 1) for _, items in launches([(2 * n, 0, 1, 93, even_slices(2 * n), 1) for n in pairs])]
    assert singles == [2 * n for n in pairs.values()]
    assert [sum(1 for i in items if i[3]) for _, items in launches([(256, 32, 8, 160, even_slices(256), 1), (16, 10, 2, 16, even_slices(16), 1)])] == [256, 32]


def test_single_key_blocks(launches):
    """Left over above whole rounds of 256 pairs: all up to 128 pairs, 64 to 208, none; 128 with slices; never halves."""
    pairs = {256: 0, 257: 1, 384: 128, 385: 64, 464: 64, 465: 0, 511: 0, 1024: 0}
    items = [i for _, i in launches([(2 * n, 0, 1, 93, even_slices(2 * n), 2) for n in pairs])]
    assert [sum(1 for i in x if i[3] == 1) for x in items] == [2 * n for n in pairs.values()] and not any(i[3] == 2 for x in items for i in x)
    assert [sum(1 for i in x if i[3]) for _, x in launches([(256, 32, 8, 160, even_slices(256), 2), (16, 10, 2, 16, even_slices(16), 2)])] == [256, 32]
