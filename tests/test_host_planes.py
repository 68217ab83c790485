"""The read-back's plane copier on the CPU (tests/host_replay/planes.cpp): any
number of pieces and slots, with and without memory for helper threads; it runs
under a C entry point, so it throws nothing.
"""
import os
import subprocess

import pytest

import test_host_replay as R


@pytest.mark.parametrize("sanitizer", ["undefined", "thread"])
def test_planes_are_copied_whole_and_nothing_is_thrown(tmp_path, sanitizer):
    if not os.path.exists(R.CXX):
        pytest.skip("no host clang++")
    exe = str(tmp_path / "planes")
    src = os.path.join(R.ROOT, "tests", "host_replay", "planes.cpp")
    subprocess.check_call([R.CXX, "-std=c++17", "-O1", "-g1", "-pthread", "-fsanitize=" + sanitizer,
                           *(["-DPLANES_NO_STARVE"] if sanitizer == "thread" else []), "-I" + R.CSRC, "-o", exe, src])
    code, out = R._run(exe, "")
    assert code == 0 and out.strip() == "identical", out
