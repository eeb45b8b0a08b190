"""The token rule's stage arithmetic, as the kernels compile it, on the host: which tokens of every stage of
every block a token sees, against the oracle's token mask.  Frames have at least 64 tokens and a stage starts
up to 96 tokens into its block, so it can start two frames behind the block's first token."""
import functools
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import build as obuild
from paper_2506_19852_amd import build as hip_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "tests", "host", "stage_rule.hip")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(hip_build.HIPCC) and shutil.which(hip_build.HIPCC) is None:
        pytest.skip("hipcc not available")
    exe = tmp_path_factory.mktemp("host") / "stage_rule"
    r = subprocess.run([hip_build.HIPCC, *hip_build.FLAGS, "--cuda-host-only", SOURCE, "-o", str(exe)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
    return str(exe)


@functools.lru_cache(maxsize=None)
def definition(frames, s, extra, sink, num, den):
    n, nv = frames * s + extra, frames * s
    want = np.ones((n, n), dtype=bool)   # text tokens see and are seen by every token
    want[:nv, :nv] = obuild.token_mask(frames, s, sink, 0, nv, np.arange(nv), num, den)
    return want


def visibility(program, *case):
    frames, s, extra = case[:3]
    n = frames * s + extra
    r = subprocess.run([program], input=" ".join(map(str, case)).encode(), stdout=subprocess.PIPE, timeout=60)
    assert r.returncode == 0, case
    return np.frombuffer(r.stdout, dtype=np.uint8).reshape(n, n).astype(bool)


@pytest.mark.parametrize("block, stage", [(64, 32), (64, 64), (128, 32), (128, 64)])
def test_every_stage_of_every_block_matches_the_definition(program, block, stage):
    cases = [(4, s, 0, 1, 1, 1) for s in range(64, 201)]
    cases += [(12, 70, 0, 1, 1, 1), (20, 65, 0, 0, 1, 1), (9, 93, 37, 1, 13, 20), (6, 79, 200, 2, 1, 2), (3, 333, 1, 1, 3, 2)]
    for frames, s, extra, sink, num, den in cases:
        want = definition(frames, s, extra, sink, num, den)
        for own_is_query in (1, 0):
            got = visibility(program, frames, s, extra, sink, num, den, block, stage, own_is_query)
            wrong = int((got != (want if own_is_query else want.T)).sum())
            assert wrong == 0, f"{wrong} wrong pairs: {frames} frames of {s} tokens + {extra}, own_is_query {own_is_query}"
