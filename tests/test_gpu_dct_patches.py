"""hb_dct_denoise at the edges of its patches: images of one tile, sides a tile beyond or short of 32 and 64, ragged last
patches in either direction, enough patches for the larger ones, tall and wide.

With threshold 0 nothing is cut and the transform gives the image back, so the image is the reference.  Bound: a sum of
16 terms of the pixels' size rounds to 16 x 2^-24 of it, which the division by the windows of a corner pixel (0.0096)
magnifies to 1e-4; elsewhere the windows are above 0.098 and it stays below 1e-5."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,H,W", [(1, 16, 16), (1, 16, 24), (2, 40, 16), (1, 24, 136), (1, 32, 72), (1, 72, 32), (3, 64, 64), (1, 200, 40),
                                   (1, 1000, 1096), (3, 1000, 1096), (1, 40, 40000), (1, 40000, 24), (6, 584, 648), (70, 136, 128)])
def test_threshold_zero_gives_the_image_back(C, H, W):
    import torch
    from paper_2512_02371_amd import hb
    gen = torch.Generator(device="cuda").manual_seed(C + H + W)
    wide = torch.full((C, H, W + 8), float("nan"), dtype=torch.float16, device="cuda")
    x = wide[:, :, :W]
    x.copy_(torch.rand((C, H, W), generator=gen, device="cuda"))
    full = torch.full((C, H, W + 3), 7.0, device="cuda")
    out = full[:, :, :W]
    ws = torch.empty(hb.hb_dct_denoise_workspace_size(C, H, W), dtype=torch.uint8, device="cuda")
    print(f"hb_dct_denoise {C}x{H}x{W}", flush=True)
    hb.hb_dct_denoise(x, out, 0.0, ws)
    err = (out.double() - x.double()).abs()
    assert float(err.max()) <= 1e-4
    assert float(err[:, 8:H - 8, 8:W - 8].max()) <= 1e-5 if min(H, W) > 16 else True
    assert bool((full[:, :, W:] == 7.0).all()), "wrote past the row end"

