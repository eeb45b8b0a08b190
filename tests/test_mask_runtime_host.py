"""The host side of the mask builds on a runtime written for the test (tests/host/mask_runtime.hip): no GPU, no kernel runs."""
import os
import shutil
import subprocess

import pytest

from paper_2506_19852_amd import build as hip_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "tests", "host", "mask_runtime.hip")
RADIAL_EHIP = -3
KERNELS = ("mask_count_kernel", "mask_lists_kernel", "mask_fill_kernel", "dense_fill_kernel", "transpose_count_kernel", "transpose_lists_kernel",
           "transpose_fill_kernel", "scan_kernel", "partition_kernel")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(hip_build.HIPCC) and shutil.which(hip_build.HIPCC) is None:
        pytest.skip("hipcc not available")
    exe = tmp_path_factory.mktemp("host") / "mask_runtime"
    r = subprocess.run([hip_build.HIPCC, *hip_build.FLAGS, "--cuda-host-only", SOURCE, "-pthread", "-o", str(exe)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]

    def run(mode):
        r = subprocess.run([str(exe), mode], stdout=subprocess.PIPE, text=True, timeout=60)
        assert r.returncode == 0, r.stdout[-3000:]
        return [line.split() for line in r.stdout.splitlines()]
    return run


def test_nothing_follows_a_refused_launch(program):
    """Each kernel of a build reads what the ones before it write: without those it would search and write by uninitialised memory."""
    kernels = set()
    for way, launch, kernel, status, after, left in program("refuse"):
        kernels.add(next(k for k in KERNELS if k in kernel))
        assert (int(status), int(after), int(left)) == (RADIAL_EHIP, 0, 0), (way, launch, kernel)
    assert kernels == set(KERNELS)


def test_builds_that_end_early_give_their_host_memory_back(program):
    """Whatever was refused before: a build copies nothing back but the counts (one copy, where the host sizes the lists by them)."""
    for way, copies in program("ended"):
        counted = way.split("-")[0] in ("radial", "banded") and "-500-" not in way
        assert int(copies) == int(counted), way


def test_builds_without_mapped_memory_copy(program):
    lines = program("unmapped")
    assert len(lines) == 14
    for way, status, copies, right in lines:
        counted = way.split("-")[0] in ("radial", "banded") and "-500-" not in way
        assert (int(status), int(copies), int(right)) == (0, 1 + counted, 1), way


def test_builds_at_a_time_have_a_slot_each_or_copy(program):
    """32 slots for 40 threads: 8 copy, each finds its own total, and the slots are free again afterwards."""
    lines = program("together")
    assert lines == [["40", "8", "0"], ["1", "0", "0"]] * 20


def test_a_slot_that_may_still_be_written_is_not_used_again(program):
    assert program("unwaited") == [["0", "3"]]
