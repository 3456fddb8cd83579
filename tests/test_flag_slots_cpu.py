"""Host logic of the pinned slots that hold the contexts' error flags, compiled with g++ and run on the
CPU (no GPU, no HIP): one page serves a context after the other, slots are distinct and cleared when
taken, pages are bounded and given back, memory lost to a device reset is not used again, threads."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_22625_amd", "csrc")
SRC = os.path.join(ROOT, "tests", "cpp", "flag_slots.cpp")


@pytest.mark.parametrize("sanitize", ["address,undefined", "thread"])
def test_flag_slots(tmp_path, sanitize):
    exe = str(tmp_path / "flag_slots")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-pthread",
                           "-fsanitize=" + sanitize, "-I", CSRC, SRC, "-o", exe])
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0")
    r = subprocess.run([exe], capture_output=True, text=True, env=env)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "flag slot checks passed" in r.stdout
