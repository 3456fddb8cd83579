"""The workspace that the structure-aware initialisation asks for (no GPU): sizes callers may have kept
stay enough, and what the kernels use fits in them (compiled with g++)."""
import os
import subprocess

import pytest

from paper_2602_22625_amd import aids

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_22625_amd", "csrc")
SRC = os.path.join(ROOT, "tests", "cpp", "sa_layout.cpp")


def test_layout_fits(tmp_path):
    exe = str(tmp_path / "sa_layout")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
                           "-fsanitize=address,undefined", "-I", CSRC, SRC, "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "sa layout checks passed" in r.stdout


# (a few pixels, columns of many rows, the usual): (H, W, bytes)
@pytest.mark.parametrize("H,W,n", [(1, 1, 1280), (5, 6, 1280), (1000, 4, 65536), (512, 512, 4211968),
                                   (2048, 2048, 67387648)])
def test_bytes_are_what_they_were(H, W, n):
    assert aids.dbmp_sa_init_workspace_bytes(H, W) == n
