"""Where hb_fir1d takes even and odd rows apart (csrc/fir1d_plan.hpp, host arithmetic, compiled here with the host's compiler)."""
import os
import random
import subprocess

import pytest

from test_gpu_fir1d import APART

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <stdio.h>
#include "fir1d_plan.hpp"
int main() {
    hb::FirCall c;
    long long ip, op;
    int even;
    c.cu = 256;
    while (scanf("%d %d %lld %lld %d %d %d", &c.H, &c.W, &ip, &op, &even, &c.ntaps, &c.anchor) == 7) {
        c.in_pitch = ip;
        c.out_pitch = op;
        c.even = even && ip % 2 == 0;
        c.lines = op % 32 == 0;
        const hb::FirPlan p = hb::fir_plan(c);
        printf("%d %d %d %d %d %d %d %d\n", p.lean, p.step, p.nk, p.nko, p.rowsteps, p.ntiles, p.run_tiles, p.nruns);
    }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "plan.cpp", d / "plan"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2512_02371_amd", "csrc"), str(src), "-o", str(exe)], check=True)

    def ask(calls):
        out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in calls), capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, l.split())) for l in out.splitlines()]
    return ask


@pytest.mark.parametrize("H,W,pitch,even,taps,anchor,lean", [
    (4095, 4095, 4095, 1, 8, 3, 1), (2047, 2047, 2047, 1, 40, 19, 1), (4095, 4095, 4095, 1, 256, 127, 1), (300, 8191, 8191, 1, 8, 3, 1), (17, 3001, 3001, 1, 100, 49, 1),
    (4096, 4096, 4096, 1, 8, 3, 0), (4096, 4096, 4096, 0, 8, 3, 1),            # even rows that start on odd pixels, too
    (6752, 32, 39, 1, 96, 0, 0), (1000, 32, 33, 1, 8, 0, 0), (2222, 331, 331, 1, 24, 11, 0), (5428, 96, 159, 1, 211, 105, 0), (200, 501, 501, 1, 200, 99, 0),     # narrow, small
    (1025, 1012, 1013, 1, 18, 8, 0), (5453, 3253, 3317, 1, 157, 78, 0), (5446, 2942, 2943, 1, 133, 66, 0), (167, 11451, 11451, 1, 50, 6, 0), (48, 31892, 31899, 1, 48, 10, 0), (34, 11867, 11867, 1, 205, 0, 0),       # a round of waves more, a third more groups
    (142, 7154, 7155, 1, 215, 107, 1), (7706, 512, 513, 1, 41, 20, 1), (4109, 465, 465, 1, 35, 17, 1), (5547, 201, 201, 1, 40, 19, 1), (6941, 256, 256, 0, 75, 37, 1), (2758, 768, 768, 0, 211, 105, 1),        # tall
    (1579, 639, 639, 1, 228, 113, 1), (68, 128, 129, 1, 132, 65, 1), (47, 3390, 3391, 1, 80, 39, 1), (323, 832, 832, 0, 40, 19, 1), (356, 1534, 1535, 1, 34, 16, 1),
])
def test_where_rows_are_taken_apart(plan, H, W, pitch, even, taps, anchor, lean):
    assert plan([(H, W, pitch, W, even, taps, anchor)])[0][0] == lean


def test_groups_and_runs_cover_the_image_once(plan):
    rng = random.Random(4)
    calls = []
    for _ in range(3000):
        H, W, taps = int(2 ** rng.uniform(0, 14)), int(2 ** rng.uniform(3, 15)), rng.randint(1, 256)
        calls.append((H, W, W + rng.choice([0, 1, 2, 7]), W + rng.choice([0, -W % 32]), rng.choice([0, 1]), taps, rng.choice([0, taps - 1, (taps - 1) // 2])))
    apart = 0
    for c, (lean, step, nk, nko, rowsteps, ntiles, run_tiles, nruns) in zip(calls, plan(calls)):
        H, W, pitch, _, _, taps, anchor = c
        starts = [32 * (g >> 1) + (g & 1) if step == 2 else 16 * g for g in range(rowsteps)]
        assert step == (2 if lean and pitch % 2 else 1)
        rows = [y for s in starts for y in range(s, s + 16 * step, step) if y < H] if rowsteps < 40 else range(H)
        assert sorted(rows) == list(range(H)), c
        assert ntiles == -(-W // 16) and run_tiles % 2 == 0 and run_tiles * nruns >= ntiles > run_tiles * (nruns - 1), c
        assert 32 * nk >= 15 + taps + (1 if lean else anchor & 1) and 32 * nko >= 31 + taps + (1 if lean else anchor & 1), c
        apart += lean
    assert apart > 100


def test_the_calls_taken_apart_on_the_gpu_are_of_every_length(plan):
    every_second = plan([(H, W, W, W, 1, T, a) for H, W, T, a in APART])
    from_odd = plan([(H, W, W + 3, W + 2, 0, T, a) for H, W, T, a in APART])
    assert all(p[0] and p[1] == 2 for p in every_second) and all(p[0] and p[1] == 1 for p in from_odd)
    assert [p[2] for p in every_second] == list(range(1, 10))
