"""hb_iir2 at the borders between its forms: one launch with products kept (runs of one to four tiles) or made again (five to eight), two
launches with short, even and long runs, signals that start on and between dwords.  Bound: the header's, 2^-24 G max|out|."""
import numpy as np
import pytest

from paper_2512_02371_amd import synth
from hbtest import up

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,T,extra", [
    (1, 2049, 0), (3, 8192, 0), (3, 8193, 0), (2, 24576, 1), (2, 24577, 0), (2, 24577, 1), (31, 24580, 1), (32, 24580, 1), (32, 32768, 0),
    (32, 32767, 0), (5, 32768, 0), (5, 32769, 1), (128, 40000, 0), (128, 40000, 1), (191, 33000, 1), (192, 33000, 1), (192, 65536, 1), (257, 5000, 0),
    (64, 131072, 0), (127, 70000, 0), (257, 32769, 0), (3, 1 << 21, 0), (400, 2000, 0), (2, 3, 1)])
@pytest.mark.parametrize("alpha,beta", [(1.6, -0.8), (1.9, -0.9025)])
def test_every_form_keeps_the_bound(orc, C, T, extra, alpha, beta):
    import torch
    from paper_2512_02371_amd import hb
    some = sorted({0, C // 2, C - 1})
    x = synth.uniform_pm1_f16(T + C, (len(some), T))
    wide = torch.full((C, T + extra), float("nan"), dtype=torch.float16, device="cuda:0")
    sig = wide[:, :T]
    sig.copy_((torch.rand((C, T), generator=torch.Generator(device="cuda").manual_seed(C), device="cuda") * 2 - 1))
    sig[some] = up(x)
    full = torch.full((C, T + 3), 7.0, device="cuda:0")
    ws = torch.full((hb.hb_iir2_workspace_size(C, T),), 0xff, dtype=torch.uint8, device="cuda:0")
    print(f"hb_iir2 {C}x{T}+{extra} ({alpha}, {beta})", flush=True)
    hb.hb_iir2(sig, full[:, :T], alpha, beta, ws)
    got = full[some].cpu().numpy().astype(np.float64)
    ref = orc.iir2(x, float(np.float32(alpha)), float(np.float32(beta)))
    bound = 2.0 ** -24 * hb.hb_iir2_abs_gain(alpha, beta, T)
    for i, c in enumerate(some):
        assert np.abs(got[i, :T] - ref[i]).max() <= max(bound * np.abs(ref[i]).max(), 2.0 ** -24), f"channel {c}"
    assert bool((full[:, T:] == 7.0).all()), "wrote past the end of a signal"
    assert bool(torch.isfinite(full).all())


@pytest.mark.parametrize("C,T", [(1, 2049), (2, 8192), (3, 12801), (1, 16384), (32, 16383), (256, 5000), (257, 16000)])
def test_running_sums_are_exact(C, T):
    """alpha = 1, beta = 0 on multiples of 2^-10: every partial sum in any order is a multiple of it below 2^14, which fp32 holds."""
    import torch
    from paper_2512_02371_amd import hb
    x = torch.randint(-1024, 1025, (C, T), generator=torch.Generator(device="cuda").manual_seed(T), device="cuda").float().div_(1024).half()
    out = torch.empty((C, T), device="cuda")
    ws = torch.full((hb.hb_iir2_workspace_size(C, T),), 0xff, dtype=torch.uint8, device="cuda")
    print(f"hb_iir2 running sum {C}x{T}", flush=True)
    hb.hb_iir2(x, out, 1.0, 0.0, ws)
    assert torch.equal(out.double().cpu(), x.double().cpu().cumsum(1))
