"""The autotuner's sizes kept for the process, on the host: a size is used again only
for launch groups of the same shape and load, and only where it fits."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1906_11195_amd", "csrc")
SRC = os.path.join(ROOT, "tests", "native", "tune_check.cpp")


def test_kept_sizes(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs g++")
    exe = str(tmp_path / "tune_check")
    subprocess.check_call([gxx, "-O1", "-std=c++17", "-Wall", "-Werror", "-I" + CSRC, SRC, "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "tune ok" in out.stdout
