"""hb_sepblur / hb_sepblur_valu against the fp64 oracle, element by element."""
import numpy as np
import pytest

from paper_2512_02371_amd import synth
from hbtest import assert_close, padded, up

pytestmark = pytest.mark.gpu

CASES = [
    # H, W, Tx, ax, Ty, ay
    (64, 64, 16, 7, 16, 7),
    (37, 53, 16, 7, 16, 7),
    (1, 1, 1, 0, 1, 0),
    (3, 200, 5, 2, 1, 0),
    (130, 300, 16, 7, 16, 7),      # several strips and row segments, ragged tail
    (100, 70, 8, 0, 2, 1),
    (70, 100, 17, 16, 17, 0),
    (90, 80, 18, 3, 18, 9),        # three row tiles in the column window
    (90, 80, 33, 32, 33, 16),
    (120, 150, 34, 10, 34, 20),    # four
    (120, 150, 50, 25, 50, 49),    # five
    (160, 96, 64, 31, 64, 32),     # maximum taps
    (160, 96, 64, 0, 64, 63),
]


def run(fn, H, W, Tx, ax, Ty, ay, pitch_extra=0):
    import torch
    from paper_2512_02371_amd import hb
    img = synth.uniform01_f16(3000 + H * 7 + W, (H, W))
    tx = synth.gaussian_taps_f16(Tx, max(Tx / 5.0, 0.5))
    ty = synth.random_taps_f16(4000 + Ty, Ty)
    d_in = up(img)
    if pitch_extra:
        _, d_in = padded(d_in, W + pitch_extra)
    obuf, out = padded(torch.zeros((H, W), dtype=torch.float32, device="cuda:0"), W + pitch_extra)
    print(f"{fn} H={H} W={W} Tx={Tx} ax={ax} Ty={Ty} ay={ay} pitch+{pitch_extra}", flush=True)
    getattr(hb, fn)(d_in, out, tx, ax, ty, ay)
    torch.cuda.synchronize()
    return img, tx, ty, out.cpu().numpy(), obuf.cpu().numpy()


@pytest.mark.parametrize("fn", ["hb_sepblur", "hb_sepblur_valu"])
@pytest.mark.parametrize("H,W,Tx,ax,Ty,ay", CASES)
def test_sepblur_matches_oracle(orc, fn, H, W, Tx, ax, Ty, ay):
    img, tx, ty, got, _ = run(fn, H, W, Tx, ax, Ty, ay)
    assert_close(got, orc.sepblur(img, tx, ax, ty, ay), f"{fn} {H}x{W}")


@pytest.mark.parametrize("Tx,ax,Ty,ay", [(17, 16, 31, 0), (16, 1, 50, 20), (18, 0, 17, 8), (31, 30, 33, 32), (49, 24, 64, 31),
                                         (64, 63, 2, 1)])
@pytest.mark.parametrize("H,W", [(15, 7), (40, 8), (1, 33), (145, 127), (128, 129), (37, 160)])
def test_sepblur_windows_over_both_row_ends(orc, H, W, Tx, ax, Ty, ay):
    """Images about as wide as a window, a strip or a workgroup's 128 columns, every filter length's kernel."""
    img, tx, ty, got, obuf = run("hb_sepblur", H, W, Tx, ax, Ty, ay, pitch_extra=1)
    assert_close(got, orc.sepblur(img, tx, ax, ty, ay), f"{H}x{W}")
    assert np.all(obuf[:, W:] == 7.0), "wrote past the row end"


@pytest.mark.parametrize("H,W,Tx,ax,Ty,ay,extra", [
    (2050, 2100, 31, 15, 31, 15, 0),    # the marching kernel, three steps a workgroup, ragged last segment and columns
    (2048, 2176, 64, 31, 64, 40, 0),    # ... whole segments inside the image
    (2050, 2100, 16, 7, 16, 8, 1),      # ... one window per tile, rows inside lines
    (1500, 3970, 50, 49, 5, 0, 3),
    (1000, 7808, 9, 4, 50, 20, 0),      # all row tiles up front: eight steps a wave for a long column filter ...
    (500, 1000, 9, 4, 50, 20, 0),       # ... four ...
    (32, 1500, 17, 8, 64, 31, 0),       # ... two
    (31, 600, 3, 1, 34, 0, 1),
    (700, 1300, 15, 6, 18, 9, 12),      # short column filter: four steps
    (3000, 4096, 9, 4, 9, 4, 0),        # eight
    (5010, 5041, 5, 2, 17, 3, 0),       # rows inside lines, but too large for the marching kernel
])
def test_sepblur_work_splits(orc, H, W, Tx, ax, Ty, ay, extra):
    """Every split of the work over steps, waves and workgroups, on bands of rows at the top, the middle and the bottom."""
    import torch
    from paper_2512_02371_amd import hb
    gen = torch.Generator(device="cuda:0").manual_seed(H + W)
    img = torch.randint(0, 2048, (H, W), generator=gen, device="cuda:0", dtype=torch.int16).float().div_(2048).half()
    tx = synth.gaussian_taps_f16(Tx, max(Tx / 5.0, 0.5))
    ty = synth.random_taps_f16(4000 + Ty, Ty)
    obuf, out = padded(torch.zeros((H, W), dtype=torch.float32, device="cuda:0"), W + extra)
    print(f"H={H} W={W} Tx={Tx} ax={ax} Ty={Ty} ay={ay} pitch+{extra}", flush=True)
    hb.hb_sepblur(img, out, tx, ax, ty, ay)
    torch.cuda.synchronize()
    for r0 in sorted({0, max(0, H // 2 - 50), max(0, H - 100)}):
        r1 = min(H, r0 + 100)
        a, b = max(0, r0 - ay), min(H, r1 + Ty - 1 - ay)      # the rows that rows r0 .. r1 - 1 read
        ref = orc.sepblur(img[a:b].cpu().numpy().view(np.uint16), tx, ax, ty, ay)
        lo, hi = r0 - a, r1 - a
        assert_close(out[r0:r1].cpu().numpy(), ref[lo:hi], f"rows {r0}..{r1}")
    assert bool((obuf[:, W:] == 7.0).all()), "wrote past the row end"


@pytest.mark.parametrize("fn", ["hb_sepblur", "hb_sepblur_valu"])
@pytest.mark.parametrize("extra", [8, 3])
def test_sepblur_pitched_layouts(orc, fn, extra):
    H, W = 50, 150
    img, tx, ty, got, obuf = run(fn, H, W, 16, 7, 16, 7, pitch_extra=extra)
    assert_close(got, orc.sepblur(img, tx, 7, ty, 7), f"{fn} pitch+{extra}")
    assert np.all(obuf[:, W:] == 7.0), "wrote past the row end"


@pytest.mark.parametrize("fn", ["hb_sepblur", "hb_sepblur_valu"])
def test_sepblur_benchmark_shape_rows_sampled_densely(orc, fn):
    """A 512-row slab of the 4096-wide benchmark image: same strip count as the full
    configuration, several row segments, compared in full."""
    import torch
    from paper_2512_02371_amd import hb
    H, W = 512, 4096
    img = synth.uniform01_f16(1002, (H, W))
    t = synth.gaussian_taps_f16(16, 3.0)
    out = torch.zeros((H, W), dtype=torch.float32, device="cuda:0")
    getattr(hb, fn)(up(img), out, t, 7, t, 7)
    torch.cuda.synchronize()
    assert_close(out.cpu().numpy(), orc.sepblur(img, t, 7, t, 7), fn)


def test_sepblur_full_benchmark_size_sampled_bands(orc):
    """The benchmark's 4096 x 4096 launch, checked on row bands: the oracle runs on a crop with 16
    rows of margin (more than the 15-row reach of the column pass), whose inner rows do not see the crop."""
    import torch
    from paper_2512_02371_amd import hb
    H = W = 4096
    img = synth.uniform01_f16(1002, (H, W))
    t = synth.gaussian_taps_f16(16, 3.0)
    out = torch.zeros((H, W), dtype=torch.float32, device="cuda:0")
    print(f"hb_sepblur {H}x{W}", flush=True)
    hb.hb_sepblur(up(img), out, t, 7, t, 7)
    torch.cuda.synchronize()
    for y0 in (0, 48, 1000, 2047, 3333, H - 80):
        lo, hi = max(y0 - 16, 0), min(y0 + 80 + 16, H)
        ref = orc.sepblur(img[lo:hi], t, 7, t, 7)
        a, b = (0 if lo == 0 else 16), (hi - lo if hi == H else hi - lo - 16)
        assert_close(out[lo + a:lo + b].cpu().numpy(), ref[a:b], f"rows {lo + a}..{lo + b}")


@pytest.mark.parametrize("H,W,Tx,ax,Ty,ay,extra", [
    (17, 128, 16, 7, 18, 3, 0), (16, 128, 16, 7, 18, 3, 0), (33, 161, 3, 1, 34, 33, 0),       # marched, and all row tiles up front
    (25, 160, 17, 0, 35, 30, 0), (24, 160, 17, 0, 35, 30, 0), (33, 70, 9, 4, 64, 0, 1), (32, 70, 9, 4, 64, 0, 1),
    (47, 16512, 16, 8, 17, 16, 0), (48, 16512, 16, 8, 17, 16, 0), (79, 16512, 5, 2, 40, 7, 0), (80, 16512, 5, 2, 64, 7, 0),
    (1024, 1792, 9, 4, 64, 31, 0), (1040, 1920, 9, 4, 64, 31, 0), (1040, 1920, 9, 4, 50, 31, 0),
    (5010, 5041, 5, 2, 17, 3, 0), (5010, 5056, 5, 2, 50, 3, 0), (5010, 5056, 5, 2, 64, 3, 0), (5010, 5042, 5, 2, 50, 3, 0),
])
def test_sepblur_one_window_marched_or_not(orc, H, W, Tx, ax, Ty, ay, extra):
    """Filters of up to 17 taps along x on either side of every line between their two kernels."""
    test_sepblur_work_splits(orc, H, W, Tx, ax, Ty, ay, extra)
