"""hb_iir2 in one launch, a workgroup per channel: the shortest and longest signals of that form, runs of one to eight tiles, a last
run that is shorter, last tiles and blocks partly filled, and the first sizes that take two launches, against the fp64
oracle.  Bound: the header's, 2^-24 times the filter's gain times the largest output (measured: up to 0.7 of it).  Pole pairs of radius
0.95 carry a state over several runs; the running sum over all of them."""
import numpy as np
import pytest

from paper_2512_02371_amd import synth
from hbtest import up

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,T", [(1, 2048), (1, 2049), (3, 2561), (2, 8192), (5, 8193), (1, 16385), (2, 24577), (3, 32768), (2, 32769),
                                 (256, 2500), (257, 2500), (128, 32769), (130, 65536), (128, 65537), (127, 40000), (3, 16384), (128, 32768)])
@pytest.mark.parametrize("alpha,beta", [(1.6, -0.8), (1.89050791, -0.9025), (-1.2, -0.9025), (1.0, 0.0)])
def test_channels_match_the_oracle(orc, C, T, alpha, beta):
    import torch
    from paper_2512_02371_amd import hb
    gain = hb.hb_iir2_abs_gain(alpha, beta, T)
    if gain > 16384:                          # a running sum this long is refused
        with pytest.raises(hb.HbError):
            hb.hb_iir2(torch.zeros((C, T), dtype=torch.float16, device="cuda:0"), torch.empty((C, T), device="cuda:0"), alpha, beta,
                       torch.empty(hb.hb_iir2_workspace_size(C, T), dtype=torch.uint8, device="cuda:0"))
        return
    x = synth.uniform_pm1_f16(T + C, (C, T))
    full = torch.full((C, T + 5), 7.0, device="cuda:0")
    out = full[:, :T]
    ws = torch.full((hb.hb_iir2_workspace_size(C, T),), 0xff, dtype=torch.uint8, device="cuda:0")
    print(f"hb_iir2 {C}x{T} ({alpha}, {beta})", flush=True)
    hb.hb_iir2(up(x), out, alpha, beta, ws)
    some = list(range(C)) if C <= 8 else sorted({0, 1, C // 3, C // 2, C - 2, C - 1})
    got = out[some].cpu().numpy().astype(np.float64)
    ref = orc.iir2(x[some], float(np.float32(alpha)), float(np.float32(beta)))          # the coefficients that the library receives
    assert (np.abs(got - ref).max(axis=1) <= 2.0 ** -24 * gain * np.abs(ref).max(axis=1)).all()
    assert bool((full[:, T:] == 7.0).all()), "wrote past the end of a signal"
