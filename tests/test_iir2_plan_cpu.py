"""Which signals hb_iir2 takes in one launch (csrc/iir2_plan.hpp, host arithmetic, compiled here with the host's compiler)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <stdio.h>
#include "iir2_plan.hpp"
int main() {
    long long C, T;
    int even;
    while (scanf("%lld %lld %d", &C, &T, &even) == 3) printf("%d\n", hb::iir_one_launch(C, (T + 511) / 512, even != 0, 256));
}
"""


@pytest.fixture(scope="module")
def one_launch(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "plan.cpp", d / "plan"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2512_02371_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    return lambda call: int(subprocess.run([str(exe)], input=" ".join(map(str, call)), capture_output=True, text=True, check=True).stdout)


# channels, samples, signals that start on whole dwords
@pytest.mark.parametrize("C,T,even,one", [
    (1, 2048, 1, 0), (1, 2049, 1, 1), (16, 32768, 1, 1), (16, 32769, 1, 0), (256, 65536, 1, 1), (257, 4096, 1, 0),
    (2, 19456, 0, 1), (2, 19457, 0, 0), (23, 24000, 0, 0), (24, 20001, 0, 0), (24, 22528, 0, 0), (24, 22529, 0, 1), (25, 22532, 0, 1), (25, 21301, 0, 0), (25, 24576, 0, 1), (25, 24577, 0, 0),
    (26, 20001, 0, 1), (31, 24576, 0, 1), (31, 24577, 0, 0), (32, 32767, 0, 1), (191, 40001, 0, 0), (192, 40001, 0, 1),
])
def test_one_launch_or_two(one_launch, C, T, even, one):
    assert one_launch((C, T, even)) == one
