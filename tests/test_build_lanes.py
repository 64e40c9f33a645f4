"""Two-lane builds keep the caller's stream order: with a HIP runtime that only
records (tests/native/build_lanes.cpp), everything a build queued on any stream comes
before what the caller queues next on its own, also when a launch fails half way.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1702_01904_amd", "csrc")
HIP_ERROR = -3  # PRISM_EHIP


@pytest.fixture(scope="module")
def lanes(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("lanes") / "build_lanes")
    cxx = shutil.which("g++") or "/opt/rocm/llvm/bin/clang++"
    cmd = [cxx, "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
           os.path.join(ROOT, "tests", "native", "build_lanes.cpp"),
           os.path.join(CSRC, "plan.cpp"), "-o", exe]
    subprocess.run(cmd, check=True, timeout=300)

    def run(n, H, f, more, fail):
        r = subprocess.run([exe, *(str(v) for v in (n, H, f, more, fail))], check=True,
                           capture_output=True, text=True, timeout=60)
        return [int(v) for v in r.stdout.split()]
    return run


# workspaces that hold all 161 beams, 41 and 8 of them (state of one: 1 MiB)
@pytest.mark.parametrize("more", [1 << 30, 40 << 20, 7 << 20])
def test_error_between_fork_and_join_still_joins(lanes, more):
    status, streams, launches, ordered = lanes(512, 12, 4, more, -1)
    assert (status, streams, ordered) == (0, 2, 1)
    for fail in (launches // 3, launches // 2, launches - 2, launches - 1):
        status, streams, queued, ordered = lanes(512, 12, 4, more, fail)
        assert (status, queued) == (HIP_ERROR, fail + 1)
        assert ordered == 1, (more, fail)
    assert streams == 2


def test_small_build_stays_on_the_callers_stream(lanes):
    status, streams, _, ordered = lanes(128, 2, 4, 1 << 24, -1)
    assert (status, streams, ordered) == (0, 1, 1)
