"""The workgroup tiles of hb_conv2d, hb_down2 and hb_up2 (csrc/toeplitz2d_tile.hpp, host arithmetic, compiled here with the
host compiler): what a wave reads of the LDS image and of the weight table lies inside what is staged and built."""
import os
import subprocess

import pytest

from test_gpu_toeplitz_tiles import CASES, output_size

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include "toeplitz2d_tile.hpp"
using namespace hb;
template <int MODE, int NK, int NW, T2Shape SHAPE>
void tile(const char* shape) {
    using G = T2Geom<MODE, NK, NW, SHAPE>;
    for (int kh = 1 + (MODE == kT2Up); kh <= HB_MAX_TAPS_CONV2D; kh += 1 + (MODE == kT2Up))
        printf("%d %d %d %s %d %d %d %d %d %d %d %d %d %d %d %d %d %d %zu %zu %zu\n", MODE, NK, NW, shape, G::kCols, G::kRows, G::kPairs, G::kStride,
               G::kPitch, G::kCopies, G::kCopy, G::kShift, G::kPad, G::kZeroRows, kh, G::steps(kh), G::srows(kh), G::tab_rows(kh),
               G::image_bytes(kh), G::lds_bytes(kh), t2_resident(G::lds_bytes(kh)));
}
int main(int argc, char** argv) {
    const char* const shapes[] = {"row", "block", "stack", "flat", "flat_pair"};
    if (argc > 1 && !strcmp(argv[1], "resample")) {       // the tile of hb_down2 or hb_up2 for each mode nk kh Ho Wo
        for (int i = 2; i + 4 < argc; i += 5)
            puts(shapes[t2_resample_tile((T2Mode)atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2]), atoi(argv[i + 3]), atoi(argv[i + 4]), 256)]);
        return 0;
    }
    if (argc > 1) {                                       // the tile of hb_conv2d for each Ho Wo kh kw pieces
        for (int i = 1; i + 4 < argc; i += 5) {
            const T2Tile t = t2_conv_tile(atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2]), (atoi(argv[i + 3]) + 30) / 16, atoi(argv[i + 4]), 256);
            printf("%s %d\n", shapes[t.shape], t.nw);
        }
        return 0;
    }
#define CONV(nk) tile<kT2Conv, nk, 1, kT2Row>("row"); tile<kT2Conv, nk, 2, kT2Row>("row"); tile<kT2Conv, nk, 4, kT2Row>("row"); tile<kT2Conv, nk, 2, kT2Flat>("flat"); tile<kT2Conv, nk, 1, kT2Block>("block"); tile<kT2Conv, nk, 2, kT2Block>("block");
    CONV(1) CONV(2) CONV(3)
#define DOWN(nk) tile<kT2Down, nk, 1, kT2Row>("row"); tile<kT2Down, nk, 1, kT2Flat>("flat"); tile<kT2Down, nk, 1, kT2FlatPair>("flat_pair"); tile<kT2Down, nk, 1, kT2Block>("block"); tile<kT2Down, nk, 1, kT2Stack>("stack");
    DOWN(2) DOWN(3) DOWN(4)
#define UP(nk) tile<kT2Up, nk, 2, kT2Row>("row"); tile<kT2Up, nk, 2, kT2Flat>("flat"); tile<kT2Up, nk, 2, kT2Block>("block");
    UP(1) UP(2)
}
"""
FIELDS = "mode nk nw shape cols rows pairs stride pitch copies copy shift pad zero_rows kh steps srows tab_rows image lds resident".split()
CONV, DOWN, UP = 0, 1, 2


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiles")
    src, exe = d / "tiles.cpp", d / "tiles"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2512_02371_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    return str(exe)


@pytest.fixture(scope="module")
def tiles(program):
    lines = subprocess.run([program], check=True, capture_output=True, text=True).stdout.splitlines()
    return [{f: v if f == "shape" else int(v) for f, v in zip(FIELDS, line.split())} for line in lines]


def test_rows_of_the_image_and_of_the_table(tiles):
    for t in tiles:
        # step s of row pair n reads staged row stride n + s, which lies in section (stride n + s) % stride
        last = max((s % t["stride"]) * t["srows"] + t["rows"] // 2 - 1 + s // t["stride"] for s in range(t["steps"]))
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


def conv_tiles(program, calls):
    out = subprocess.run([program] + [str(int(v)) for c in calls for v in c], check=True, capture_output=True, text=True).stdout.split()
    return list(zip(out[::2], map(int, out[1::2])))


def resample_tiles(program, calls):
    return subprocess.run([program, "resample"] + [str(v) for c in calls for v in c], check=True, capture_output=True, text=True).stdout.split()


def test_widest_conv2d_tile_only_where_it_is_the_fastest(program):
    """Not where a quarter of its 256 columns would be empty, nor for rows that start on 64-byte pieces, nor tall kernels."""
    calls = [(ho, wo, k, k, True) for wo in (65, 100, 128, 129, 258, 600) for ho in (30000, 200000, 1000000) for k in (3, 32)]
    calls += [(ho, wo, k, k, False) for ho, wo in ((4096, 4096), (3464, 3456), (2880, 3056), (8192, 8192)) for k in (3, 24, 28, 32)]
    calls += [(4095, 4095, 30, 30, True), (3464, 3457, 19, 19, True), (1500, 5985, 19, 19, True), (3000, 2977, 3, 3, True)]
    assert all(t != ("row", 4) for t in conv_tiles(program, calls))
    calls = [(4095, 4095, 29, 29, True), (8000, 1985, 3, 3, True), (3464, 3457, 18, 18, True), (1500, 5985, 1, 1, True)]
    assert conv_tiles(program, calls) == [("row", 4)] * 4


def test_narrow_images_take_the_conv2d_tile_that_they_fill(program):
    """None that is twice as wide as the image, whatever its height."""
    calls = [(ho, wo, k, k, pieces) for wo in (1, 8, 16, 31, 32, 33, 48, 57, 64) for ho in (1, 16384, 16385, 65408, 65409, 1000000) for k in (1, 16, 32) for pieces in (0, 1)]
    for (ho, wo, _, _, _), tile in zip(calls, conv_tiles(program, calls)):
        assert tile == (("block", 1) if wo <= 32 and ho > 256 * 64 else ("block", 2) if wo > 56 and ho > 511 * 128 else ("row", 1))


def test_outputs_of_few_rows_take_the_flat_tile(program):
    flat = [(16, 80000, 32, 32, False), (48, 80000, 32, 32, False), (96, 40000, 32, 32, False), (80, 70000, 32, 32, False), (48, 98305, 3, 3, True)]
    tall = [(34, 88000, 32, 32, False), (16, 32000, 32, 32, False), (64, 80000, 32, 32, False), (97, 300000, 32, 32, False), (48, 98304, 3, 3, False)]
    assert [shape for shape, _ in conv_tiles(program, flat + tall)] == ["flat"] * 5 + ["row"] * 5
    # hb_down2 and hb_up2: mode, chunks of the window, kernel rows, Ho, Wo
    flat = [(DOWN, 2, 16, 32, 24577), (DOWN, 3, 25, 32, 24577), (DOWN, 3, 3, 48, 49153), (DOWN, 4, 30, 80, 49153), (DOWN, 4, 30, 32, 32769),
            (UP, 2, 32, 48, 49153), (UP, 2, 4, 96, 49153), (UP, 1, 4, 63, 49153), (UP, 1, 4, 32, 65537), (UP, 2, 4, 1, 49153)]
    pair = [(DOWN, 3, 26, 32, 24577), (DOWN, 4, 31, 32, 32769)]
    tall = [(DOWN, 3, 16, 33, 24577), (DOWN, 3, 16, 49, 300000), (DOWN, 3, 16, 81, 300000), (DOWN, 3, 16, 32, 24576), (DOWN, 4, 16, 32, 32768),
            (DOWN, 3, 26, 33, 300000), (UP, 2, 4, 63, 300000), (UP, 1, 4, 64, 300000), (UP, 1, 4, 97, 300000), (UP, 1, 4, 32, 65536)]
    assert resample_tiles(program, flat + pair + tall) == ["flat"] * 10 + ["flat_pair"] * 2 + ["row"] * 10


def test_narrow_outputs_of_the_resampling_stages(program):
    calls = [(mode, 3 if mode == DOWN else 1, 16, ho, wo) for mode in (DOWN, UP) for ho in (16384, 16385, 1 << 20) for wo in (1, 16, 17, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161)]
    for (mode, _, _, ho, wo), shape in zip(calls, resample_tiles(program, calls)):
        narrow = ("stack" if wo <= 16 else "block" if wo <= 160 and (wo - 1) % 64 < 32 else "row") if mode == DOWN else "block" if wo <= 64 else "row"
        assert shape == (narrow if ho > 256 * 64 else "row"), (mode, ho, wo)


def test_flat_tiles_fit_a_compute_unit_twice(tiles):
    """Those of hb_down2 and hb_up2, four waves or, above 25 kernel rows (30 with more than 18 taps across) of hb_down2, two."""
    for t in tiles:
        if t["mode"] == UP and t["shape"] == "flat" or t["mode"] == DOWN and t["shape"] == ("flat_pair" if t["kh"] > (30 if t["nk"] == 4 else 25) else "flat"):
            assert t["resident"] >= 2, t


def test_gpu_cases_reach_every_tile(program, tiles):
    """The cases of test_gpu_toeplitz_tiles.py take the tiles that they name, and all there are."""
    reached = set()
    for op, H, W, kh, kw, extra, tile in CASES:
        Ho, Wo = output_size(op, H, W)
        if op == "conv2d":
            nk, got = (30 + kw) // 16, "%s %d" % conv_tiles(program, [(Ho, Wo, kh, kw, (Wo + extra) % 16 != 0)])[0]
        else:
            nk = (45 + kw) // 16 if op == "down2" else 1 if kw <= 18 else 2
            got = resample_tiles(program, [(DOWN if op == "down2" else UP, nk, kh, Ho, Wo)])[0]
        assert got == tile, (op, H, W, kh, kw, got)
        reached.add((op, nk, tile))
    names = {CONV: "conv2d", DOWN: "down2", UP: "up2"}
    assert reached == {(names[t["mode"]], t["nk"], f"{t['shape']} {t['nw']}" if t["mode"] == CONV else t["shape"]) for t in tiles}
