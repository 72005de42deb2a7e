"""hb_iir2 in one launch, a workgroup per channel: the shortest and longest signals of that form, runs of one to eight tiles, a last
run that is shorter, last tiles and blocks partly filled, and the first sizes that take two launches, against the fp64
oracle.  Bound: 2^-23 per step (products of two fp16 parts, sums of 32) magnified by the filter's gain, as for the other
forms."""
import numpy as np
import pytest

from paper_2512_02371_amd import synth
from hbtest import up

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,T", [(1, 2048), (1, 2049), (3, 2561), (2, 8192), (5, 8193), (1, 16385), (2, 24577), (3, 32768), (2, 32769),
                                 (256, 2500), (257, 2500), (128, 32769), (130, 65536), (128, 65537), (127, 40000)])
def test_channels_match_the_oracle(orc, C, T):
    import torch
    from paper_2512_02371_amd import hb
    alpha, beta = 1.6, -0.8
    x = synth.uniform_pm1_f16(T + C, (C, T))
    full = torch.full((C, T + 5), 7.0, device="cuda:0")
    out = full[:, :T]
    ws = torch.full((hb.hb_iir2_workspace_size(C, T),), 0xff, dtype=torch.uint8, device="cuda:0")
    print(f"hb_iir2 {C}x{T}", flush=True)
    hb.hb_iir2(up(x), out, alpha, beta, ws)
    some = sorted({0, C // 2, C - 1})
    got, ref = out[some].cpu().numpy().astype(np.float64), orc.iir2(x[some], alpha, beta)
    gain = hb.hb_iir2_abs_gain(alpha, beta, T)
    assert np.abs(got - ref).max() <= 4 * 2.0 ** -23 * gain * np.abs(ref).max()
    assert bool((full[:, T:] == 7.0).all()), "wrote past the end of a signal"
