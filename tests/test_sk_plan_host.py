"""How SK sweeps are cut into launches, on the host: every sweep is run, recomputations
fall between launches, and neither the blocks nor the accepted flips of a launch pass
the kernels' 32-bit counters, whatever the recompute period."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1906_11195_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include "sg_sk_plan.h"
int main()
{
    const long periods[] = {1, 64, 1 << 20, 0x7fffffffL};
    const int blocks[] = {1, 2, 64, 512};
    const long wanted[] = {1, 1000, (1L << 32) - 1};
    for (long period : periods)
        for (int nb : blocks)
            for (long n : wanted) {
                if (n > 1000 && period < (1 << 20)) continue;   // (many launches)
                long t = 5, left = n;
                while (left > 0) {
                    const long to_check = period - t % period;
                    const long k = sg::sk_launch_sweeps(left, to_check, nb);
                    if (k < 1 || k > left || k > to_check) return 1;
                    if (k > 0x7fffffffL / nb) return 2;
                    if ((unsigned long)k * nb * 64 > 0xffffffffUL) return 3;
                    t += k;
                    left -= k;
                }
            }
    std::puts("launches ok");
    return 0;
}
"""


def test_launches_stay_within_the_counters(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs g++")
    src, exe = str(tmp_path / "plan.cpp"), str(tmp_path / "plan")
    with open(src, "w") as f:
        f.write(DRIVER)
    subprocess.check_call([gxx, "-O1", "-std=c++17", "-I" + CSRC, src, "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and "launches ok" in out.stdout, out.returncode
