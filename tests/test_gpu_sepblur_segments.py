"""The march of hb_sepblur at every rule for the length of its segments: rows of whole, half and quarter lines, input rows on and between
dwords, one to five row tiles, from a workgroup per unit to where all take eight steps.  The vector twin is the reference; both round the
row pass to fp16, from sums in another order, so that a value below 1 may come out one fp16 unit apart, 2^-11."""
import pytest

from paper_2512_02371_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,pad,extra", [
    (500, 1000, 0, 0), (1079, 1917, 0, 0), (1800, 1808, 0, 0), (1801, 1811, 0, 0), (1801, 1811, 1, 0), (2700, 1500, 0, 0), (2048, 2048, 0, 8),
    (2048, 2048, 0, 0), (2300, 2300, 0, 0), (2000, 3000, 0, 0), (2401, 2603, 0, 0), (2160, 3840, 0, 0), (1500, 6000, 0, 0), (3000, 3000, 0, 0),
    (2750, 3333, 0, 0), (3300, 3300, 0, 0), (3600, 3600, 0, 0), (3584, 3616, 0, 0), (3001, 4001, 0, 0), (4000, 4002, 0, 2)])
@pytest.mark.parametrize("Tx,Ty", [(5, 5), (40, 17), (16, 33), (31, 18), (48, 49), (64, 64)])
def test_segments(H, W, pad, extra, Tx, Ty):
    import torch
    from paper_2512_02371_amd import hb
    gen = torch.Generator(device="cuda").manual_seed(H + W)
    x = torch.full((H, W + pad), float("nan"), dtype=torch.float16, device="cuda")[:, :W]
    x.copy_(torch.rand((H, W), generator=gen, device="cuda"))
    full = torch.full((H, W + extra), 7.0, device="cuda")
    want = torch.empty((H, W), device="cuda")
    tx, ty = synth.gaussian_taps_f16(Tx, 3.0 * Tx / 16), synth.gaussian_taps_f16(Ty, 3.0 * Ty / 16)
    print(f"hb_sepblur {H}x{W}+{pad} to +{extra} {Tx}x{Ty}", flush=True)
    hb.hb_sepblur(x, full[:, :W], tx, Tx // 2, ty, Ty // 3)
    hb.hb_sepblur_valu(x, want, tx, Tx // 2, ty, Ty // 3)
    # the column taps are positive and sum to about one, so no more than that reaches an output (and 2^-24 a step of the sums)
    assert float((full[:, :W] - want).abs().max()) <= 2.0 ** -11 * 1.01
    assert bool((full[:, W:] == 7.0).all()), "wrote past the row end"
