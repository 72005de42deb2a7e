"""hb_conv2d, hb_down2, hb_up2 at the edges of their workgroup tiles and of the rules that choose among them, against the
fp64 oracle."""
import numpy as np
import pytest

from paper_2512_02371_amd import synth
from hbtest import assert_close, padded, up

pytestmark = pytest.mark.gpu

CASES = [
    # op, H, W, kh, kw (anchors in the middle); sizes are of the input
    ("conv2d", 64, 64, 3, 2),            # one narrow tile (64 x 64), whole ...
    ("conv2d", 65, 193, 32, 31),         # ... and one past it
    ("conv2d", 63, 127, 31, 1),
    ("conv2d", 16512, 32, 32, 32),       # the tile for narrow images (32 x 128), whole ...
    ("conv2d", 16385, 31, 17, 31),       # ... and ragged, with one wave of four at work in the last
    ("conv2d", 20500, 9, 3, 2),
    ("conv2d", 20500, 33, 16, 2),        # many tiles of 64 x 64: narrow images of more columns ...
    ("conv2d", 10300, 160, 3, 17),       # ... and ones that would leave half of a 128-wide tile empty
    ("conv2d", 1280, 2048, 2, 17),       # the middle tile (64 x 128), its first size, whole tiles
    ("conv2d", 1281, 2051, 3, 3),        # ... and ragged
    ("conv2d", 49, 130817, 3, 2),        # the wide tile (64 x 256): rows that start inside lines ...
    ("conv2d", 49, 130848, 28, 2),       # ... and many kernel rows
    ("conv2d", 48, 98337, 3, 2),         # few rows, many columns: 48 rows are the most ...
    ("conv2d", 49, 98337, 2, 3),         # ... and this one is too many
    ("conv2d", 16, 98560, 7, 17),        # whole short tiles
    ("conv2d", 17, 98305, 32, 5),
    ("down2", 128, 128, 16, 16),         # one tile of outputs (64 x 64), whole ...
    ("down2", 130, 131, 32, 32),         # ... and past it; the taps share the image's LDS
    ("down2", 126, 126, 15, 2),
    ("down2", 64, 98306, 3, 4),          # the short tile and the last height that takes it
    ("down2", 65, 98306, 4, 3),
    ("down2", 31, 98816, 17, 18),
    ("down2", 32770, 64, 3, 2),          # narrow and tall: the block of 32 x 128 outputs, whole columns ...
    ("down2", 33023, 45, 17, 16),        # ... and ragged ones
    ("down2", 32899, 130, 32, 31),
    ("down2", 33280, 32, 2, 2),          # ... and the stack of 16 x 256
    ("down2", 32769, 17, 31, 18),
    ("down2", 33791, 8, 32, 32),
    ("up2", 8256, 32, 32, 32),           # ... and the block of 64 x 128
    ("up2", 8193, 31, 4, 18),
    ("down2", 63, 66001, 30, 32),        # few rows, many taps: the flat tile of four waves ...
    ("down2", 64, 65664, 31, 31),        # ... and of two, whole ...
    ("down2", 33, 65601, 32, 19),
    ("down2", 17, 49301, 26, 18),        # ... and with fewer taps across
    ("down2", 95, 98433, 25, 5),
    ("up2", 32, 64, 16, 16),             # one tile of outputs (64 x 128), whole ...
    ("up2", 33, 65, 32, 32),             # ... and past it
    ("up2", 31, 63, 2, 18),
    ("up2", 16, 49153, 4, 6),            # the short tile and the last height that takes it
    ("up2", 17, 49153, 6, 4),
    ("up2", 8, 49408, 20, 2),
    ("conv2d", 57, 256, 3, 3),           # whole columns, rows missing from the last tile: vector stores of some rows ...
    ("conv2d", 1281, 2176, 5, 32),
    ("down2", 126, 256, 3, 18),
    ("up2", 17, 128, 6, 6),
    ("down2", 4098, 8192, 2, 2),         # ... through the L2 (more than 32 MB of output, rows off the 128-byte lines: pitch below)
]


@pytest.mark.parametrize("op,H,W,kh,kw", CASES)
def test_tile_edges(orc, op, H, W, kh, kw):
    import torch
    from paper_2512_02371_amd import hb
    img = synth.uniform01_f16(H + W, (H, W))
    k = synth.random_kernel2d_f16(kh * 33 + kw, kh, kw)
    Ho, Wo = {"conv2d": (H, W), "down2": ((H + 1) // 2, (W + 1) // 2), "up2": (2 * H, 2 * W)}[op]
    n = 2 if op == "up2" else 1                            # phases per axis: hb_up2 anchors among kh / 2
    ay, ax = (kh // n - 1) // 2, (kw // n - 1) // 2
    pitch = (Wo + 31) // 32 * 32 if kh == 28 else Wo + 1 if H == 4098 else Wo
    obuf, out = padded(torch.zeros((Ho, Wo), dtype=torch.float32, device="cuda:0"), pitch)
    print(f"{op} {H}x{W} {kh}x{kw}", flush=True)
    getattr(hb, "hb_" + op)(up(img), out, k, ay, ax)
    torch.cuda.synchronize()
    assert_close(out.cpu().numpy(), getattr(orc, op)(img, k, ay, ax), f"{op} {H}x{W} {kh}x{kw}")
    assert bool((obuf[:, Wo:] == 7.0).all()), "wrote past the row end"
