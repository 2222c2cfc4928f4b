"""Workspace of the weight gradients: its size, fixed by max_batch, against the
partial sums of every batch up to max_batch (host arithmetic of
wgrad_chunks.hpp, compiled here)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2102_00514_amd", "csrc")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ is not available")
    exe = str(tmp_path_factory.mktemp("chunks") / "wgrad_chunks_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, "-o", exe,
                    os.path.join(HERE, "host_build", "wgrad_chunks_check.cpp")], check=True)
    return exe


@pytest.mark.parametrize("width", (1, 20, 128, 150, 256, 1024))
@pytest.mark.parametrize("lpos, columns, rows", ((16, 16, 20), (4, 64, 80), (64, 4, 5), (12, 32, 40), (128, 8, 10)))
def test_no_batch_exceeds_the_workspace(check, width, lpos, columns, rows):
    res = subprocess.run([check, str(width), str(lpos), str(columns), str(rows), "4096"], check=True,
                         capture_output=True, text=True)
    over, more, uncovered = map(int, res.stdout.split())
    assert over == 0 and uncovered == 0
    if (width, lpos) == (128, 16):
        assert more > 0    # the chunks of max_batch alone would not bound them
