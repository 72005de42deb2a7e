"""The workgroup tiles of hb_conv2d, hb_down2 and hb_up2 (csrc/toeplitz2d_tile.hpp, host arithmetic, compiled here with the
host compiler): what a wave reads of the LDS image and of the weight table lies inside what is staged and built."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <stdio.h>
#include "toeplitz2d_tile.hpp"
using namespace hb;
template <int MODE, int NK, int NW, bool SHORT>
void tile(const char* shape) {
    using G = T2Geom<MODE, NK, NW, SHORT>;
    for (int kh = 1 + (MODE == kT2Up); kh <= HB_MAX_TAPS_CONV2D; kh += 1 + (MODE == kT2Up))
        printf("%d %d %d %s %d %d %d %d %d %d %d %d %d %d %d %d %d %d %zu %zu %zu\n", MODE, NK, NW, shape, G::kCols, G::kRows, G::kPairs, G::kStride,
               G::kPitch, G::kCopies, G::kCopy, G::kShift, G::kPad, G::kZeroRows, kh, G::steps(kh), G::srows(kh), G::tab_rows(kh),
               G::image_bytes(kh), G::lds_bytes(kh), t2_resident(G::lds_bytes(kh)));
}
int main() {
#define CONV(nk) tile<kT2Conv, nk, 1, false>("row"); tile<kT2Conv, nk, 2, false>("row"); tile<kT2Conv, nk, 4, false>("row"); tile<kT2Conv, nk, 2, true>("short");
    CONV(1) CONV(2) CONV(3)
#define DOWN(nk) tile<kT2Down, nk, 1, false>("row"); tile<kT2Down, nk, 1, true>("short");
    DOWN(2) DOWN(3) DOWN(4)
#define UP(nk) tile<kT2Up, nk, 2, false>("row"); tile<kT2Up, nk, 2, true>("short");
    UP(1) UP(2)
}
"""
FIELDS = "mode nk nw shape cols rows pairs stride pitch copies copy shift pad zero_rows kh steps srows tab_rows image lds resident".split()
CONV, DOWN, UP = 0, 1, 2


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiles")
    src, exe = d / "tiles.cpp", d / "tiles"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2512_02371_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()
    return [{f: v if f == "shape" else int(v) for f, v in zip(FIELDS, line.split())} for line in lines]


def test_rows_of_the_image_and_of_the_table(tiles):
    for t in tiles:
        # step s of row pair n reads staged row stride n + s, which lies in section (stride n + s) % stride
        last = max((s % t["stride"]) * t["srows"] + t["pairs"] - 1 + s // t["stride"] for s in range(t["steps"]))
        assert (last + 1) * t["pitch"] * 2 <= t["image"], t
        # of the weight table, step s reads row s + row0
        if t["mode"] == UP:
            rows = [4 * s + 2 * dy + dx for s in range(t["steps"]) for dy in (0, 1) for dx in (0, 1)]
        else:
            rows = [t["zero_rows"] - (1 + (t["mode"] == DOWN)) * dy + s for s in range(t["steps"]) for dy in (0, 1)]
        assert min(rows) == 0 and max(rows) == t["tab_rows"] - 1, t      # all that is built is read, and nothing else


def test_runs_of_the_table(tiles):
    for t in tiles:
        for m in range(16):
            for h in range(2):
                t0 = 8 * h - {CONV: m, DOWN: 2 * m, UP: m // 2}[t["mode"]] + t["pad"]
                copy = t0 // t["shift"] % t["copies"]
                start = t0 - t["shift"] * copy
                assert t0 % t["shift"] == 0 and start >= 0 and start % (t["shift"] * t["copies"]) == 0, t
                assert start + 16 * (t["nk"] - 1) + 8 <= t["copy"], t


def test_general_conv2d_tile_has_three_workgroups_per_compute_unit(tiles):
    """As many as its registers allow, up to the largest kernel (two zero rows of the table too many made it two from 31
    kernel rows on)."""
    general = [t for t in tiles if (t["mode"], t["nw"], t["shape"]) == (CONV, 2, "row")]
    assert len(general) == 96 and all(t["resident"] >= 3 for t in general), [(t["nk"], t["kh"], t["lds"]) for t in general if t["resident"] < 3]
