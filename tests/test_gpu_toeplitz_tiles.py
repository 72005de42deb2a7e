"""hb_conv2d, hb_down2, hb_up2 at the edges of their workgroup tiles and of the rules that choose among them, against the
fp64 oracle."""
import numpy as np
import pytest

from paper_2512_02371_amd import synth
from hbtest import assert_close, padded, up

pytestmark = pytest.mark.gpu

CASES = [
    # op, H, W, kh, kw (anchors in the middle), pitch beyond the output's width, tile; sizes are of the input.  The tiles are those
    # of csrc/toeplitz2d_tile.hpp on 256 compute units (test_toeplitz_tiles_cpu.py checks them): waves and, for hb_conv2d, 16-column
    # tiles per wave.  Every tile with every number of window chunks (hb_conv2d: up to 1, 17, 32 taps across; hb_down2: 2, 18,
    # 32; hb_up2: 18, 32).
    ("conv2d", 64, 64, 3, 2, 0, "row 1"),                # 64 x 64, whole ...
    ("conv2d", 65, 193, 32, 31, 0, "row 1"),             # ... and one past it
    ("conv2d", 63, 127, 31, 1, 0, "row 1"),
    ("conv2d", 20500, 33, 16, 2, 0, "row 1"),            # many of them: narrow images ...
    ("conv2d", 10300, 160, 16, 17, 0, "row 1"),          # ... and ones that would leave half of 128 columns empty ...
    ("conv2d", 10300, 161, 15, 3, 0, "row 2"),           # ... unless their rows start inside 64-byte pieces
    ("conv2d", 1280, 2048, 2, 17, 0, "row 2"),           # 64 x 128, its first size, whole tiles
    ("conv2d", 1281, 2051, 3, 3, 0, "row 2"),            # ... and ragged
    ("conv2d", 1281, 2176, 5, 32, 0, "row 2"),           # ... whole columns, rows missing from the last tile
    ("conv2d", 57, 41216, 30, 1, 0, "row 2"),
    ("conv2d", 50, 147473, 3, 2, 0, "row 4"),            # 64 x 256: rows that start inside pieces ...
    ("conv2d", 50, 147473, 2, 1, 0, "row 4"),
    ("conv2d", 128, 73985, 18, 18, 0, "row 4"),          # ... and whole rows of tiles
    ("conv2d", 50, 147473, 2, 3, 15, "row 2"),           # ... rows that start on pieces
    ("conv2d", 49, 130817, 3, 2, 0, "row 2"),
    ("conv2d", 49, 130848, 28, 2, 0, "row 2"),
    ("conv2d", 16512, 32, 32, 32, 0, "block 1"),         # narrow images (128 x 32), whole ...
    ("conv2d", 16385, 31, 17, 31, 0, "block 1"),         # ... and ragged, with one wave of four at work in the last
    ("conv2d", 20500, 9, 3, 2, 0, "block 1"),
    ("conv2d", 16999, 8, 7, 1, 0, "block 1"),
    ("conv2d", 65536, 64, 7, 18, 0, "block 2"),          # ... and 128 x 64 where they fill that
    ("conv2d", 65430, 61, 16, 2, 0, "block 2"),
    ("conv2d", 65537, 57, 3, 1, 0, "block 2"),
    ("conv2d", 48, 98337, 3, 2, 0, "flat 2"),            # few rows, many columns: 48 rows are the most ...
    ("conv2d", 49, 98337, 2, 3, 0, "row 2"),             # ... and this one is too many
    ("conv2d", 16, 98560, 7, 17, 0, "flat 2"),           # whole flat tiles
    ("conv2d", 17, 98305, 32, 5, 0, "flat 2"),
    ("conv2d", 3, 98400, 3, 1, 0, "flat 2"),
    ("conv2d", 17, 41001, 20, 18, 0, "flat 2"),          # many taps: from fewer columns on
    ("conv2d", 5, 41472, 32, 32, 31, "flat 2"),
    ("conv2d", 66, 70001, 8, 3, 0, "flat 2"),
    ("down2", 128, 128, 16, 16, 0, "row"),               # 64 x 64 outputs, whole ...
    ("down2", 130, 131, 32, 32, 0, "row"),               # ... and past it; the taps share the image's LDS
    ("down2", 126, 126, 15, 2, 0, "row"),
    ("down2", 126, 256, 3, 18, 0, "row"),                # whole columns, rows missing
    ("down2", 4098, 8192, 2, 2, 1, "row"),               # ... through the L2: over 32 MB of output, rows off the 128-byte lines
    ("down2", 32770, 64, 3, 2, 0, "block"),              # narrow and tall: 128 x 32, whole columns ...
    ("down2", 33023, 45, 17, 16, 0, "block"),            # ... and ragged ones
    ("down2", 32899, 130, 32, 31, 0, "block"),
    ("down2", 33280, 32, 2, 2, 0, "stack"),              # 256 x 16
    ("down2", 32769, 17, 31, 18, 0, "stack"),
    ("down2", 33791, 8, 32, 32, 0, "stack"),
    ("down2", 64, 98306, 3, 4, 0, "flat"),               # few rows, many columns ...
    ("down2", 65, 98304, 4, 3, 0, "row"),                # ... and one row too many, up to this width
    ("down2", 65, 98306, 4, 3, 0, "flat"),
    ("down2", 31, 98816, 17, 18, 0, "flat"),
    ("down2", 1, 49400, 5, 2, 0, "flat"),
    ("down2", 95, 98433, 25, 5, 0, "flat"),
    ("down2", 63, 66001, 30, 32, 0, "flat"),             # ... many taps: four waves ...
    ("down2", 64, 65664, 31, 31, 0, "flat_pair"),        # ... and two, whole ...
    ("down2", 33, 65601, 32, 19, 0, "flat_pair"),
    ("down2", 17, 49301, 26, 18, 0, "flat_pair"),        # ... and with fewer taps across
    ("down2", 33, 49300, 27, 2, 0, "flat_pair"),
    ("up2", 32, 64, 16, 16, 0, "row"),                   # 64 x 128 outputs, whole ...
    ("up2", 33, 65, 32, 32, 0, "row"),                   # ... and past it
    ("up2", 31, 63, 2, 18, 0, "row"),
    ("up2", 17, 128, 6, 6, 0, "row"),                    # whole columns, rows missing
    ("up2", 8256, 32, 32, 32, 0, "block"),               # narrow and tall: 128 x 64
    ("up2", 8193, 31, 4, 18, 0, "block"),
    ("up2", 16, 49153, 4, 6, 0, "flat"),                 # few rows, many columns
    ("up2", 16, 32768, 4, 6, 0, "row"),                  # ... and one column too few
    ("up2", 17, 49153, 6, 4, 0, "flat"),
    ("up2", 8, 49408, 20, 2, 0, "flat"),
    ("up2", 1, 24601, 32, 32, 0, "flat"),
    ("up2", 48, 24700, 2, 20, 0, "flat"),
]


def output_size(op, H, W):
    return {"conv2d": (H, W), "down2": ((H + 1) // 2, (W + 1) // 2), "up2": (2 * H, 2 * W)}[op]


@pytest.mark.parametrize("op,H,W,kh,kw,extra,tile", CASES)
def test_tile_edges(orc, op, H, W, kh, kw, extra, tile):
    import torch
    from paper_2512_02371_amd import hb
    img = synth.uniform01_f16(H + W, (H, W))
    k = synth.random_kernel2d_f16(kh * 33 + kw, kh, kw)
    Ho, Wo = output_size(op, H, W)
    n = 2 if op == "up2" else 1                            # phases per axis: hb_up2 anchors among kh / 2
    ay, ax = (kh // n - 1) // 2, (kw // n - 1) // 2
    pitch = Wo + extra
    obuf, out = padded(torch.zeros((Ho, Wo), dtype=torch.float32, device="cuda:0"), pitch)
    print(f"{op} {H}x{W} {kh}x{kw} {tile}", flush=True)
    getattr(hb, "hb_" + op)(up(img), out, k, ay, ax)
    torch.cuda.synchronize()
    assert_close(out.cpu().numpy(), getattr(orc, op)(img, k, ay, ax), f"{op} {H}x{W} {kh}x{kw}")
    assert bool((obuf[:, Wo:] == 7.0).all()), "wrote past the row end"
