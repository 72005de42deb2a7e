"""Outputs of more than 32 MB whose rows break 16-byte pieces or start inside 128-byte lines: they are stored through the L2,
not past it.  Inputs are drawn on the GPU; the oracle sees bands of rows."""
import numpy as np
import pytest

from paper_2512_02371_amd import synth
from hbtest import assert_close, padded

pytestmark = pytest.mark.gpu


def image(seed, H, W):
    import torch
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    return torch.randint(0, 2048, (H, W), generator=gen, device="cuda:0", dtype=torch.int16).float().div_(2048).half()


def bits(t):
    return t.cpu().numpy().view(np.uint16)


@pytest.mark.parametrize("H,W,extra", [(2901, 2899, 0), (2900, 2898, 3), (8705, 1001, 0), (4200, 4203, 1), (2050, 16390, 0)])
def test_sat2d(orc, H, W, extra):
    import torch
    from paper_2512_02371_amd import hb
    img = image(H, H, W)
    obuf, out = padded(torch.zeros((H, W), dtype=torch.float32, device="cuda:0"), W + extra)
    ws = torch.empty(hb.hb_sat2d_workspace_size(H, W), dtype=torch.uint8, device="cuda:0")
    print(f"sat2d {H}x{W} pitch+{extra}", flush=True)
    hb.hb_sat2d(img, out, ws)
    torch.cuda.synchronize()
    assert_close(out.cpu().numpy(), orc.sat2d(bits(img)), f"{H}x{W}")
    assert bool((obuf[:, W:] == 7.0).all()), "wrote past the row end"


@pytest.mark.parametrize("H,W,kh,kw,ay,ax,extra", [(5802, 5798, 4, 6, 1, 3, 0), (5801, 5803, 17, 3, 8, 0, 1), (700, 50001, 32, 32, 5, 30, 2)])
def test_down2(orc, H, W, kh, kw, ay, ax, extra):
    import torch
    from paper_2512_02371_amd import hb
    img, Ho, Wo = image(H, H, W), (H + 1) // 2, (W + 1) // 2
    assert Ho * Wo * 4 > 32 << 20
    taps = synth.random_kernel2d_f16(kh, kh, kw)
    obuf, out = padded(torch.zeros((Ho, Wo), dtype=torch.float32, device="cuda:0"), Wo + extra)
    print(f"down2 {H}x{W} {kh}x{kw} pitch+{extra}", flush=True)
    hb.hb_down2(img, out, taps, ay, ax)
    torch.cuda.synchronize()
    for r0 in (0, Ho // 2 - 10, Ho - 20):
        r1 = r0 + 20
        a = max(0, 2 * r0 - ay) & ~1                          # the rows that rows r0 .. r1 - 1 read, from an even one on
        b = min(H, 2 * (r1 - 1) + kh - ay)
        ref = orc.down2(bits(img[a:b]), taps, ay, ax)
        assert_close(out[r0:r1].cpu().numpy(), ref[r0 - a // 2:r1 - a // 2], f"rows {r0}..{r1}")
    assert bool((obuf[:, Wo:] == 7.0).all()), "wrote past the row end"


@pytest.mark.parametrize("H,W,kh,kw,ay,ax,extra", [(1451, 1451, 4, 6, 1, 2, 0), (1450, 1453, 16, 2, 7, 0, 1), (300, 15001, 32, 32, 5, 15, 3)])
def test_up2(orc, H, W, kh, kw, ay, ax, extra):
    import torch
    from paper_2512_02371_amd import hb
    img = image(H, H, W)
    assert 4 * H * W * 4 > 32 << 20
    taps = synth.random_kernel2d_f16(kh, kh, kw)
    obuf, out = padded(torch.zeros((2 * H, 2 * W), dtype=torch.float32, device="cuda:0"), 2 * W + extra)
    print(f"up2 {H}x{W} {kh}x{kw} pitch+{extra}", flush=True)
    hb.hb_up2(img, out, taps, ay, ax)
    torch.cuda.synchronize()
    for r0 in (0, H // 2 - 5, H - 10):                        # input rows
        r1 = r0 + 10
        a, b = max(0, r0 - ay), min(H, r1 - 1 + kh // 2 - ay)
        ref = orc.up2(bits(img[a:b]), taps, ay, ax)
        assert_close(out[2 * r0:2 * r1].cpu().numpy(), ref[2 * (r0 - a):2 * (r1 - a)], f"rows {r0}..{r1}")
    assert bool((obuf[:, 2 * W:] == 7.0).all()), "wrote past the row end"
