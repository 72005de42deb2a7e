"""hb_fir1d's long filters at the rules for the number of runs: one or two waves per SIMD by the alignment of the rows and the size, and
three for images of a few rows.  Pixels 0 or 1 and taps of k / 256: sums of either order are exact in fp32, so the vector
twin is matched bit for bit."""
import numpy as np
import pytest

from paper_2512_02371_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,pad,extra", [
    (2040, 2056, 0, 0), (2040, 2058, 0, 0), (2056, 2050, 0, 3), (2056, 2051, 0, 0), (2056, 2051, 1, 0), (2048, 2048, 0, 32), (2890, 2904, 0, 0),
    (4500, 4660, 0, 0), (4500, 4662, 0, 0), (8, 100000, 0, 0), (15, 60001, 0, 2), (1, 300000, 0, 0), (16, 70000, 0, 0), (1000, 4200, 6, 1)])
@pytest.mark.parametrize("T", [34, 90, 100, 176, 177, 256])
def test_runs(H, W, pad, extra, T):
    import torch
    from paper_2512_02371_amd import hb
    gen = torch.Generator(device="cuda").manual_seed(H + W)
    x = torch.full((H, W + pad), float("nan"), dtype=torch.float16, device="cuda")[:, :W]
    x.copy_(torch.rand((H, W), generator=gen, device="cuda") < 0.4)
    taps = synth.f64_to_f16_bits(np.random.default_rng(T).integers(1, 64, T) / 256.0)
    full, want = torch.full((H, W + extra), 7.0, device="cuda"), torch.empty((H, W), device="cuda")
    print(f"hb_fir1d {H}x{W}+{pad} to +{extra} T={T}", flush=True)
    hb.hb_fir1d(x, full[:, :W], taps, T // 3)
    hb.hb_fir1d_valu(x, want, taps, T // 3)
    assert torch.equal(full[:, :W], want)
    assert bool((full[:, W:] == 7.0).all()), "wrote past the row end"
