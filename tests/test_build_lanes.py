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
    status, streams, launches, ordered, apart, once = lanes(512, 12, 4, more, -1)
    assert (apart, once) == (1, 1)
    assert (status, streams, ordered) == (0, 2, 1)
    for fail in (launches // 3, launches // 2, launches - 2, launches - 1):
        status, streams, queued, ordered, apart, _ = lanes(512, 12, 4, more, fail)
        assert (status, queued) == (HIP_ERROR, fail + 1)
        assert (ordered, apart) == (1, 1), (more, fail)
    assert streams == 2


# little in all; much in all, but in passes shorter than a launch
@pytest.mark.parametrize("n,H,f", [(128, 2, 4), (128, 300, 2)])
def test_small_passes_stay_on_the_callers_stream(lanes, n, H, f):
    status, streams, _, ordered, apart, once = lanes(n, H, f, 1 << 24, -1)
    assert (status, streams, ordered, apart, once) == (0, 1, 1, 1, 1)


# 161, 97, 49 and 5 beams on workspaces for 1 wave up to more than all of them
@pytest.mark.parametrize("n,H,f", [(512, 4, 4), (768, 12, 8), (1024, 12, 16), (2048, 12, 128)])
def test_lanes_stay_inside_the_workspace(lanes, n, H, f):
    wave = 8 * n * (n // 2)
    for waves in (*range(1, 12), 23, 24, 25, 47, 48, 49, 50, 96, 97, 98, 160, 161, 162, 200):
        status, streams, _, ordered, apart, once = lanes(n, H, f, (waves - 1) * wave, -1)
        assert (status, ordered, apart, once) == (0, 1, 1, 1), waves
        assert streams == (1 if waves == 1 else 2), waves
