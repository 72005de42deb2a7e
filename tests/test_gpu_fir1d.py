"""hb_fir1d / hb_fir1d_valu against the fp64 oracle, element by element."""
import numpy as np
import pytest

from paper_2512_02371_amd import synth
from hbtest import assert_close, padded, up

pytestmark = pytest.mark.gpu

CASES = [
    # H, W, T, anchor
    (256, 256, 8, 3),        # the benchmark configuration
    (37, 53, 8, 3),          # ragged in both directions, narrower than one tile
    (1, 1, 1, 0),            # degenerate
    (5, 7, 5, 4),
    (130, 300, 16, 7),       # several tiles plus a ragged tail
    (64, 200, 16, 0),        # the paper's left-anchored form
    (33, 129, 64, 63),
    (33, 129, 64, 0),
    (48, 96, 33, 16),
    (16, 70, 17, 1),
    # the large-tap regime: 4 to 9 windows of 32 pixels per tile, fewer tiles per strip
    (40, 700, 100, 50),
    (40, 700, 128, 0),
    (33, 640, 129, 128),
    (20, 1000, 200, 99),
    (48, 1200, 256, 127),    # maximum taps
    (17, 600, 256, 255),     # rightmost anchor
    (17, 600, 256, 0),
    (9, 250, 256, 100),      # narrower than one window
    (20, 7, 33, 3),          # narrower than eight pixels: falls to the vector-ALU kernel
    (17, 8, 17, 16),
    (18, 9, 256, 0),         # every window reaches over both ends of the row
    (3, 65, 16, 15),         # one pixel past a strip
    (2100, 90, 200, 3),      # one run of six tiles per row group
    (31, 4100, 40, 39),      # many runs of four tiles, the last one short
    (800, 2603, 100, 50),    # runs as long as the windows ahead of them
    (3, 70001, 20, 3),       # few rows: four waves per SIMD
    (1, 120000, 200, 199),   # ... two, of longer runs
    (100, 100, 159, 80),     # narrow, rows inside lines: the vector-ALU kernel
    (100, 128, 159, 80),     # narrow, whole lines: walked
]


def run(fn, H, W, T, a, pitch_extra=0, offset=0, seed=0):
    import torch
    from paper_2512_02371_amd import hb
    img = synth.uniform01_f16(1000 + seed + H * 7 + W, (H, W))
    taps = synth.random_taps_f16(2000 + seed + T, T)
    d_in = up(img)
    if pitch_extra or offset:
        base = torch.full((H, W + pitch_extra + offset), 3.0, dtype=torch.float16, device="cuda:0")
        base[:, offset:offset + W] = d_in
        d_in = base[:, offset:offset + W]
    obuf, out = padded(torch.zeros((H, W), dtype=torch.float32, device="cuda:0"), W + pitch_extra)
    print(f"{fn} H={H} W={W} T={T} a={a} pitch+{pitch_extra} off={offset}", flush=True)
    getattr(hb, fn)(d_in, out, taps, a)
    torch.cuda.synchronize()
    return img, taps, out.cpu().numpy(), obuf.cpu().numpy()


@pytest.mark.parametrize("fn", ["hb_fir1d", "hb_fir1d_valu"])
@pytest.mark.parametrize("H,W,T,a", CASES)
def test_fir1d_matches_oracle(orc, fn, H, W, T, a):
    img, taps, got, _ = run(fn, H, W, T, a)
    assert_close(got, orc.fir1d(img, taps, a), f"{fn} {H}x{W} T={T} a={a}")


@pytest.mark.parametrize("extra", [1, 4, 7, 20])
@pytest.mark.parametrize("H,W,T,a", [(19, 500, 40, 20), (40, 31, 100, 3), (17, 130, 256, 255), (5, 1040, 64, 0)])
def test_fir1d_long_filters_with_rows_inside_lines(orc, H, W, T, a, extra):
    """Row pitches that move the rows' starts through a 128-byte line, runs that end inside one."""
    img, taps, got, obuf = run("hb_fir1d", H, W, T, a, pitch_extra=extra)
    assert_close(got, orc.fir1d(img, taps, a), f"{H}x{W} T={T} pitch+{extra}")
    assert np.all(obuf[:, W:] == 7.0), "wrote past the row end"


@pytest.mark.parametrize("fn", ["hb_fir1d", "hb_fir1d_valu"])
@pytest.mark.parametrize("extra,offset", [(8, 0), (3, 0), (5, 1), (12, 8)])
def test_fir1d_pitched_and_misaligned_layouts(orc, fn, extra, offset):
    H, W, T, a = 40, 150, 8, 3
    img, taps, got, obuf = run(fn, H, W, T, a, pitch_extra=extra, offset=offset)
    assert_close(got, orc.fir1d(img, taps, a), f"{fn} pitch+{extra} off {offset}")
    assert np.all(obuf[:, W:] == 7.0), "wrote past the row end"


def test_fir1d_long_filter_at_blur_size(orc):
    """256 taps on a 512-row slab of a 4096-wide image (the width of the blur benchmark)."""
    img, taps, got, _ = run("hb_fir1d", 512, 4096, 256, 127, seed=9)
    assert_close(got, orc.fir1d(img, taps, 127), "256 taps, 512 x 4096")


@pytest.mark.parametrize("fn", ["hb_fir1d", "hb_fir1d_valu"])
def test_fir1d_impulse_and_constant(fn):
    """Invariants that need no oracle: mirrored taps, tap sum."""
    import torch
    from paper_2512_02371_amd import hb
    T, a, H, W = 8, 3, 20, 100
    taps = synth.random_taps_f16(5, T)
    k = synth.f16_bits_to_f64(taps)
    img = np.zeros((H, W))
    img[7, 50] = 1.0
    out = torch.zeros((H, W), dtype=torch.float32, device="cuda:0")
    getattr(hb, fn)(up(synth.f64_to_f16_bits(img)), out, taps, a)
    got = out.cpu().numpy()
    for x in range(W):
        r = 50 - x + a
        assert got[7, x] == (np.float32(k[r]) if 0 <= r < T else 0.0)
    getattr(hb, fn)(up(synth.f64_to_f16_bits(np.full((H, W), 0.5))), out, taps, a)
    assert np.allclose(out.cpu().numpy(), 0.5 * k.sum(), atol=1e-6)


@pytest.mark.parametrize("T,a", [(20, 19), (64, 0)])
def test_fir1d_large_image_of_whole_lines(orc, T, a):
    """More runs per row where the image is large, on bands of rows."""
    import torch
    from paper_2512_02371_amd import hb
    H, W = 5030, 5024
    gen = torch.Generator(device="cuda:0").manual_seed(T)
    img = torch.randint(0, 2048, (H, W), generator=gen, device="cuda:0", dtype=torch.int16).float().div_(2048).half()
    out = torch.zeros((H, W), dtype=torch.float32, device="cuda:0")
    taps = synth.random_taps_f16(T, T)
    hb.hb_fir1d(img, out, taps, a)
    for r0 in (0, 2512, H - 30):
        ref = orc.fir1d(img[r0:r0 + 30].cpu().numpy().view(np.uint16), taps, a)
        assert_close(out[r0:r0 + 30].cpu().numpy(), ref, f"rows {r0}..")


@pytest.mark.parametrize("H,W,T,a", [(17, 201, 3, 1), (18, 64, 16, 0), (33, 333, 17, 3), (96, 97, 17, 4), (97, 129, 18, 17), (16, 90, 8, 3),
                                     (384, 1031, 48, 2), (383, 1027, 48, 3), (400, 1001, 49, 11), (31, 515, 100, 99), (32, 515, 160, 1),
                                     (193, 2051, 255, 0), (200, 2001, 256, 100), (79, 701, 256, 99)])
@pytest.mark.parametrize("extra,offset", [(0, 0), (1, 0), (2, 1), (27, 4)])
def test_fir1d_even_and_odd_rows_apart(orc, H, W, T, a, extra, offset):
    """Rows that start on odd pixels, every second one or all of them, around the groups of 32 rows and the windows' room."""
    img, taps, got, obuf = run("hb_fir1d", H, W, T, a, pitch_extra=extra, offset=offset)
    assert_close(got, orc.fir1d(img, taps, a), f"{H}x{W} T={T} pitch+{extra} off {offset}")
    assert np.all(obuf[:, W:] == 7.0), "wrote past the row end"


# calls whose odd rows are taken apart, one to nine windows (tests/test_fir1d_plan_cpu.py holds the library to that)
APART = [(64, 33, 12, 5), (61, 1777, 36, 3), (161, 1055, 80, 19), (68, 113, 100, 50), (33, 49, 130, 64), (60, 333, 160, 80), (200, 1991, 200, 99), (300, 1401, 230, 100), (200, 1971, 256, 128)]


@pytest.mark.parametrize("H,W,T,a", APART)
@pytest.mark.parametrize("extra,offset", [(0, 0), (2, 1)])
def test_fir1d_rows_apart_of_every_length(orc, H, W, T, a, extra, offset):
    img, taps, got, obuf = run("hb_fir1d", H, W, T, a, pitch_extra=extra, offset=offset)
    assert_close(got, orc.fir1d(img, taps, a), f"{H}x{W} T={T} pitch+{extra} off {offset}")
    assert np.all(obuf[:, W:] == 7.0), "wrote past the row end"
