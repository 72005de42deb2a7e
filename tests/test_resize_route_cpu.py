"""Which kernels a call of hb_resize takes (csrc/resize_route.hpp, host arithmetic, compiled here with the host's compiler)."""
import os
import random
import subprocess

import pytest

from test_gpu_resize import APART_OWN, APART_SHARED, NOT_APART

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <stdio.h>
#include "resize_route.hpp"
int main() {
    hb::RzCall c;
    int even, lines;
    long long pitch;
    c.cu = 256;
    while (scanf("%d %d %d %d %d %d %d %lld %d %d", &c.C, &c.H, &c.W, &c.Ho, &c.Wo, &c.band_y, &c.band_x, &pitch, &even, &lines) == 10) {
        c.in_pitch = pitch;
        c.even = even;
        c.lines = lines;
        const hb::RzRoute r = hb::rz_route(c);
        printf("%d %d %d\n", r.one_launch, r.apart, r.groups);
    }
}
"""


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    d = tmp_path_factory.mktemp("route")
    src, exe = d / "route.cpp", d / "route"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2512_02371_amd", "csrc"), str(src), "-o", str(exe)], check=True)

    def ask(calls):
        lines = []
        for C, H, W, Ho, Wo, pitch, even in calls:
            by, bx = (6 * n // m + 1 if m <= n else 6 for n, m in ((H, Ho), (W, Wo)))
            lines.append(f"{C} {H} {W} {Ho} {Wo} {by} {bx} {pitch} {even} 0")
        out = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, l.split())) for l in out.splitlines()]
    return ask


TWO, PLAIN, APART = "two launches", "one launch", "one launch, even and odd rows apart"


@pytest.mark.parametrize("call,want", [
    # groups of 16 output rows that need more rows than a wave's T holds: nothing is read apart
    ((16, 2048, 2048, 228, 228, 2049), TWO), ((3, 4000, 4001, 444, 2667, 4001), TWO), ((1, 8191, 8191, 910, 910, 8191), TWO),
    ((3, 4095, 4095, 500, 500, 4095), TWO), ((16, 1277, 1311, 180, 86, 1311), TWO),
    # nor where most windows reach over the row's ends, or three workgroups to a unit are a round more than four
    ((16, 3012, 89, 1799, 60, 89), PLAIN), ((16, 5140, 115, 506, 8, 115), PLAIN), ((1, 1266, 1483, 876, 1026, 1483), PLAIN),
    ((1, 8191, 1001, 120, 200, 1001), PLAIN), ((2, 217, 2189, 198, 176, 2189), PLAIN), ((3, 5998, 439, 4068, 297, 439), PLAIN),
    ((8, 2048, 2048, 227, 227, 2049), APART), ((8, 2048, 2048, 512, 512, 2049), APART), ((1, 4095, 4095, 900, 900, 4095), APART),
    # a round more in large images or with several chunks a window; shared groups with more than one to a unit
    ((8, 787, 5325, 164, 7830, 5389), APART), ((8, 3907, 465, 659, 78, 465), APART), ((16, 473, 4430, 60, 4397, 4495), PLAIN), ((1, 1611, 2997, 1803, 1624, 2997), APART),
    ((1, 586, 2559, 67, 4036, 2559), APART), ((16, 4295, 284, 271, 17, 285), PLAIN), ((1, 603, 5703, 425, 448, 5767), PLAIN), ((16, 4166, 311, 5190, 35, 311), PLAIN), ((3, 3632, 1409, 545, 145, 1409), TWO), ((1, 1101, 5825, 70, 6899, 5825), TWO),
    ((1, 1947, 6281, 214, 690, 6281), APART), ((3, 1912, 2923, 671, 1025, 2923), APART), ((8, 1265, 5731, 221, 1001, 5731), APART),
])
def test_routes_of_odd_pitches(route, call, want):
    (one, apart, _), = route([call + (0,)])
    assert (APART if apart else PLAIN if one else TWO) == want


def test_rows_are_read_apart_only_where_the_kernel_can(route):
    rng = random.Random(3)
    calls = []
    while len(calls) < 4000:
        C = rng.choice([1, 1, 2, 3, 8, 16])
        H, W = (int(2 ** rng.uniform(4, 13.5)) for _ in "HW")
        Ho, Wo = (max(1, int(n / 2 ** rng.uniform(-1, 5))) for n in (H, W))
        pitch = W + rng.choice([0, 0, 1, 2, 64])
        if max(H // Ho, W // Wo) <= 85:
            calls.append((C, H, W, Ho, Wo, pitch, 0 if pitch % 2 else rng.choice([0, 1])))
    taken = 0
    for c, (one, apart, groups) in zip(calls, route(calls)):
        C, H, W, Ho, Wo, pitch, even = c
        assert groups in (0, 1, 2, 4)
        if not apart:
            continue
        assert pitch % 2 == 1, c
        taken += one
        by, bx = (6 * n // m + 1 if m <= n else 6 for n, m in ((H, Ho), (W, Wo)))
        rows = (min(16 * max(groups, 1), Ho) - 1) * H / Ho + by
        assert rows <= (160 if groups else 512), c
        assert (min(16, Wo) - 1) * W / Wo + bx + 2 <= 32 * 12, c
    assert taken > 100


def test_the_parity_tests_run_what_they_say(route):
    for calls, want in ((APART_SHARED, lambda one, apart, groups: one and apart and groups == 0), (APART_OWN, lambda one, apart, groups: one and apart and groups > 0),
                        (NOT_APART, lambda one, apart, groups: not apart)):
        for call in calls:
            one, apart, groups = route([call + (call[2] + 1 + call[2] % 2, 0)])[0]
            assert want(one, apart, groups), (call, one, apart, groups)
    assert {route([c + (c[2] + 2, 0)])[0][2] for c in APART_OWN} == {1, 2, 4}
    assert {route([c + (c[2] + 2, 0)])[0][0] for c in NOT_APART} == {0, 1}
