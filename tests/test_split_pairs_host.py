"""The planner's split in two of the costliest units, on the host: used where sizes
spread over decades leave no leading group, not where it shortens nothing, and
within the budget and the chunks a unit has."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1906_11195_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <vector>
#include "sg_split_plan.h"
int main(int, char** argv)
{
    int budget = 0, n = 0;
    long share = 0;
    if (std::scanf("%d %ld %d", &budget, &share, &n) != 3) return 2;
    std::vector<sg::SplitUnit> u(n);
    for (auto& x : u) {
        long c = 0, cap = 0;
        int res = 0;
        if (std::scanf("%ld %d %ld", &c, &res, &cap) != 3) return 2;
        x = sg::SplitUnit{c, res != 0, cap};
    }
    std::vector<int> m;
    std::printf("%d", sg::plan_split(u, share, budget, 0, m));
    for (int x : m) std::printf(" %d", x);
    std::printf("\n");
    return 0;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("plan")
    src, exe = str(d / "plan.cpp"), str(d / "plan")
    with open(src, "w") as f:
        f.write(DRIVER)
    subprocess.check_call([gxx, "-O1", "-std=c++17", "-I" + CSRC, src, "-o", exe])

    def run(budget, units):
        share = sum(c for c, _, _ in units) // 256
        text = "%d %d %d\n" % (budget, share, len(units)) + "\n".join("%d %d %d" % u for u in units)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=60, check=True).stdout.split()
        return int(out[0]), [int(x) for x in out[1:]]

    return run


SPREAD = [(int(11 * 2.0 ** (20 - 10 * i / 300)), 0, 40) for i in range(300)]


@pytest.mark.parametrize("budget,pairs", [(64, 32), (33, 16), (24, 12)])
def test_costliest_units_in_two(plan, budget, pairs):
    used, m = plan(budget, SPREAD)
    assert used == 2 * pairs and m == [2] * pairs + [1] * (300 - pairs)


def test_units_left_whole(plan):
    assert plan(8, SPREAD)[0] == 0                                     # the fifth is as long as the first
    assert plan(64, [(8000000, 0, 40)] * 64)[0] == 0                   # equal: nothing gets shorter
    assert plan(64, [(c, 1, 40) for c, _, _ in SPREAD])[0] == 0        # resident
    assert plan(64, [(c, 0, 1) for c, _, _ in SPREAD])[0] == 0         # no chunks for two


BLOCKS = r"""
#include <cstdio>
#include "sg_split_plan.h"
int main()
{
    for (int slots : {1, 2, 4}) {
        if (sg::split_chunk_blocks(slots, 1, 512) != 2 || sg::split_chunk_blocks(slots, 1 << 20, 1) != 2) return 1;
    }
    // 16 wavefronts: one block up to 31 chunks of two blocks in the largest class
    if (sg::split_chunk_blocks(8, 1, 16) != 1 || sg::split_chunk_blocks(8, 31 * 128, 16) != 1) return 2;
    if (sg::split_chunk_blocks(8, 31 * 128 + 1, 16) != 2 || sg::split_chunk_blocks(8, 1 << 20, 16) != 2) return 3;
    std::puts("blocks ok");
    return 0;
}
"""


def test_blocks_of_split_chunks(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs g++")
    src, exe = str(tmp_path / "blocks.cpp"), str(tmp_path / "blocks")
    with open(src, "w") as f:
        f.write(BLOCKS)
    subprocess.check_call([gxx, "-O1", "-std=c++17", "-I" + CSRC, src, "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and "blocks ok" in out.stdout, out.returncode
