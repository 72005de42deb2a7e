"""Which kernel takes the filters of one window in hb_sepblur (csrc/sepblur_plan.hpp, compiled here with the host's compiler)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <stdio.h>
#include "sepblur_plan.hpp"
int main() {
    int H, W, nt, even, lines;
    while (scanf("%d %d %d %d %d", &H, &W, &nt, &even, &lines) == 5) printf("%d\n", hb::sep_marches({H, W, nt, even != 0, lines != 0, 256}));
}
"""


@pytest.fixture(scope="module")
def marches(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "plan.cpp", d / "plan"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2512_02371_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    return lambda call: int(subprocess.run([str(exe)], input=" ".join(map(str, call)), capture_output=True, text=True, check=True).stdout)


# rows, columns, taps down, even input rows, whole lines of the output
@pytest.mark.parametrize("H,W,taps,even,lines,march", [
    (256, 256, 16, 1, 1, 1), (1024, 1024, 45, 1, 1, 1), (4096, 4096, 16, 1, 1, 1), (2047, 2045, 45, 0, 0, 1), (8191, 8191, 16, 0, 0, 1), (200, 32, 64, 1, 1, 1),
    (8192, 8192, 16, 1, 1, 0), (16, 16, 64, 1, 0, 0), (28, 288, 44, 1, 1, 0), (29, 24, 41, 0, 0, 0), (31, 28, 49, 0, 0, 0), (32, 102, 41, 0, 0, 1), (33, 300000, 16, 1, 1, 0),
    (12872, 159, 41, 1, 0, 0), (10773, 32, 55, 1, 1, 0), (8629, 192, 22, 1, 1, 0), (14921, 149, 19, 1, 1, 0),         # tall and narrow
    (11097, 444, 57, 1, 0, 1), (5177, 129, 49, 1, 0, 1), (12157, 448, 54, 1, 1, 1),                                    # of more pixels, lower
    (14921, 149, 19, 1, 0, 1), (14921, 149, 19, 0, 1, 1), (900, 159, 41, 1, 0, 1),                                     # inside lines with few row tiles, odd rows, few workgroups
    (84, 27920, 50, 1, 1, 0), (84, 27920, 50, 0, 0, 1), (41, 44110, 58, 1, 0, 0), (52, 22311, 64, 0, 0, 0), (26, 31499, 37, 0, 0, 0), (30, 18989, 45, 0, 0, 0), (56, 31936, 27, 1, 1, 0), (46, 31144, 49, 1, 1, 0),      # long rows
])
def test_where_the_march_is_the_slower_one(marches, H, W, taps, even, lines, march):
    assert marches((H, W, (taps + 30) // 16, even, lines)) == march
