"""The walk of hb_fir1d's long filters at every count of windows that the even and the odd tiles of a pair need, at the least
and the most taps of each, with either parity of the anchor: runs of few and of many pairs, odd counts of tiles, the
last pair and the last tile partly outside.  Pixels 0 or 1 and taps of k / 256: sums of either order are exact in fp32, so the
oracle is matched bit for bit."""
import numpy as np
import pytest

from paper_2512_02371_amd import synth
from hbtest import padded, up

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("edge", [18, 33, 34, 49])            # taps + (anchor & 1) - 32 (nk - 2): the least and most for nk, nk and nk, nk + 1
@pytest.mark.parametrize("nk", [2, 3, 4, 5, 6, 7, 8, 9])
def test_pairs_of_tiles(orc, nk, edge):
    import torch
    from paper_2512_02371_amd import hb
    rng = np.random.default_rng(100 * nk + edge)
    for odd in (0, 1):
        T = min(edge + 32 * (nk - 2) - odd, 256)
        taps = synth.f64_to_f16_bits(rng.integers(1, 64, T) / 256.0)
        anchor = 2 * int(rng.integers(0, (T - odd + 1) // 2)) + odd
        assert (anchor & 1) == odd and 0 <= anchor < T
        for H, W, extra in ((5, 20 * nk + 9, 0), (21, 1037, 3), (33, 608, 32), (18, 16, 0), (250, 2090, 0)):
            img = synth.binary01_f16(nk * W + H, (H, W))
            _, x = padded(up(img), W + extra)
            buf, out = padded(torch.zeros((H, W), device="cuda:0"), W + extra)
            print(f"hb_fir1d {H}x{W}+{extra} T={T} anchor={anchor}", flush=True)
            hb.hb_fir1d(x, out, taps, anchor)
            got = out.cpu().numpy().astype(np.float64)
            assert np.array_equal(got, orc.fir1d(img, taps, anchor)), (H, W, T, anchor)
            assert bool((buf[:, W:] == 7.0).all()), "wrote past the row end"
