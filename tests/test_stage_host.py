"""How the words of a measurement come to host memory, checked on the host: the
header is compiled with g++ into a small driver with a stand-in for the device."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1906_11195_amd", "csrc")
SRC = os.path.join(ROOT, "tests", "native", "stage_check.cpp")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("stage") / "stage_check")
    subprocess.check_call([gxx, "-O1", "-std=c++17", "-Wall", "-Werror", "-pthread", "-I" + CSRC, SRC, "-o", exe])

    def run(what):
        out = subprocess.run([exe, what], capture_output=True, text=True, timeout=120)
        assert out.returncode == 0, out.stdout + out.stderr
        assert "stage ok" in out.stdout

    return run


def test_segments_past_2_to_32_words(check):
    check("large")


def test_multispin_states_are_one_range(check):
    check("states")


def test_copies_without_mapped_memory(check):
    check("plain")


def test_words_in_pieces(check):
    check("pieces")


def test_pool_of_mapped_memory_is_bounded(check):
    check("pool")
