"""The token rule as a wave of 32 tokens applies it to the stages of its list, on the host: the element masks against the oracle's token
mask, and the stages said to be seen wholly or not at all against the masks.  Frames of 64 to 200 tokens (waves and stages in
two frames, blocks in three), ragged ends, text, sinks, width scales."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import patterns as op
from paper_2506_19852_amd import build as hip_build
from tests.test_token_rule_host import definition, visibility

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "tests", "host", "list_rule.hip")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(hip_build.HIPCC) and shutil.which(hip_build.HIPCC) is None:
        pytest.skip("hipcc not available")
    exe = tmp_path_factory.mktemp("host") / "list_rule"
    r = subprocess.run([hip_build.HIPCC, *hip_build.FLAGS, "--cuda-host-only", SOURCE, "-o", str(exe)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
    return str(exe)


@pytest.mark.parametrize("block, stage", [(64, 32), (64, 64), (128, 32), (128, 64)])
def test_masks_of_every_wave_and_stage_match_the_definition(program, block, stage):
    cases = [(4, s, 0, 1, 1, 1) for s in range(64, 201)]
    cases += [(12, 70, 0, 1, 1, 1), (20, 65, 0, 0, 1, 1), (9, 93, 37, 1, 13, 20), (6, 79, 200, 2, 1, 2), (3, 333, 1, 1, 3, 2), (70, 64, 0, 0, 1, 2)]
    for frames, s, extra, sink, num, den in cases:
        if frames * s > 2000 and (block, stage) != (64, 64):
            continue  # the sub-sampled diagonals (64 frames apart) once
        want = definition(frames, s, extra, sink, num, den)
        for own_is_query in (1, 0):
            got = visibility(program, frames, s, extra, sink, num, den, block, stage, own_is_query, 0)
            wrong = int((got != (want if own_is_query else want.T)).sum())
            assert wrong == 0, f"{wrong} wrong pairs: {frames} frames of {s} tokens + {extra}, own_is_query {own_is_query}"


@pytest.mark.parametrize("block, stage", [(64, 32), (64, 64), (128, 32), (128, 64)])
def test_masks_of_banded_patterns_match_the_definition(program, block, stage):
    """Half widths of nothing, the diagonal, some positions and the whole frame, as the mask build hands them to the kernels (its
    table ends with an entry for the frame after the last)."""
    for frames, s, sink in ((5, 64, 0), (6, 100, 1), (7, 131, 2), (4, 200, 0), (9, 77, 1)):
        widths = [(s, -1, 0, s - 1, 5, 40, s // 2, -1, 63)[(d * 5 + s) % 9] for d in range(frames)]
        want = op.banded_mask_rows(frames, s, sink, widths, np.arange(frames * s))
        for own_is_query in (1, 0):
            got = visibility(program, frames, s, 0, sink, 1, 1, block, stage, own_is_query, frames + 1, *widths, -1)
            wrong = int((got != (want if own_is_query else want.T)).sum())
            assert wrong == 0, f"{wrong} wrong pairs: {frames} frames of {s} tokens, half widths {widths}, own_is_query {own_is_query}"
