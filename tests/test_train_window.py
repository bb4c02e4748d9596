"""The trainer's window of chunks (paper_2304_09409_amd/csrc/train_window.h): how many operand blocks it
allocates for a frame, and how far it goes down when memory is short. Host logic only, checked by a small C++
program over need, room and what is allocated."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2304_09409_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_window_sizes(tmp_path):
    exe = str(tmp_path / "train_window_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I" + CSRC, os.path.join(HERE, "train_window_check.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "window ok" in r.stdout
