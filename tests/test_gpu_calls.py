"""The native marshalling of calls: what it takes gives what ctypes gives, and what it does not take is left to ctypes."""
import numpy as np
import pytest

from paper_2512_02371_amd import hb, synth
from hbtest import up

pytestmark = pytest.mark.gpu

H, W = 40, 70


def usual(torch):
    """Entry point -> (arguments of a usual call, its output)."""
    img = up(synth.uniform01_f16(1, (H, W)))
    f32 = lambda *s: torch.zeros(s, dtype=torch.float32, device="cuda:0")
    ws = lambda n: torch.empty(n, dtype=torch.uint8, device="cuda:0")
    k2, g = synth.random_kernel2d_f16(2, 6, 4), synth.gaussian_taps_f16(7, 2.0)
    x, w = up(synth.uniform_pm1_f16(3, (1, 20, 24, 64))), up(synth.normal_f16(4, (3, 3, 64, 64), 1.0 / 24.0))
    sy, cy = hb.hb_lanczos3_matrix(H, 17)
    sx, cx = hb.hb_lanczos3_matrix(W, 30)
    c = {}
    c["fir1d"] = [img, f32(H, W), synth.random_taps_f16(5, 9), 4], 1
    c["conv2d"] = [img, f32(H, W), k2, 2, 1], 1
    c["down2"] = [img, f32(H // 2, W // 2), k2, 2, 1], 1
    c["up2"] = [img, f32(2 * H, 2 * W), k2, 1, 1], 1
    c["sepblur"] = [img, f32(H, W), g, 3, g, 3], 1
    c["sat2d"] = [img, f32(H, W), ws(hb.hb_sat2d_workspace_size(H, W))], 1
    c["conv3x3"] = [x, w, torch.zeros_like(x)], 2
    c["pyr_level"] = [img, f32(H, W), torch.zeros((H // 2, W // 2), dtype=torch.float16, device="cuda:0")], 1
    c["resize"] = [img[None], f32(1, 17, 30), ws(hb.hb_resize_workspace_size(1, H, 30)), torch.from_numpy(sy).cuda(), up(cy),
                   torch.from_numpy(sx).cuda(), up(cx)], 1
    c["iir2"] = [img, f32(H, W), 1.2, -0.5, ws(hb.hb_iir2_workspace_size(H, W))], 1
    c["dct_denoise"] = [up(synth.uniform01_f16(6, (2, 24, 40))), f32(2, 24, 40), 0.1, ws(hb.hb_dct_denoise_workspace_size(2, 24, 40))], 1
    return c


@pytest.mark.parametrize("name", ["fir1d", "conv2d", "down2", "up2", "sepblur", "sat2d", "conv3x3", "pyr_level", "resize", "iir2", "dct_denoise"])
def test_usual_calls_are_taken_and_equal_ctypes(name, monkeypatch):
    import torch
    hb.load()
    args, o = usual(torch)[name]
    call = getattr(hb._calls, name)
    print(name, flush=True)
    # On the current stream: its products take a millisecond each, and what the call reads is written behind them.  On the default
    # stream it would read zeros.
    image, busy = args[0].clone(), torch.zeros((2, 8192, 8192), dtype=torch.float16, device="cuda:0")
    args[0].zero_()
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        for _ in range(3):
            torch.mm(busy[0], busy[0], out=busy[1])
        args[0].copy_(image)
        assert call(*args) is True
    stream.synchronize()
    got = args[o].clone()
    args[o].zero_()
    entry = getattr(hb, "hb_" + name)
    with monkeypatch.context() as m:
        m.setattr(hb, "_calls", None)
        assert entry(*args) is args[o]
    assert torch.equal(got, args[o])
    args[o].zero_()
    assert entry(*args) is args[o] and torch.equal(got, args[o])

    class Sub(torch.Tensor):
        pass
    from torch.overrides import TorchFunctionMode

    class Watch(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    args[o].zero_()
    for i in (0, 1):
        other = list(args)
        other[i] = args[i].as_subclass(Sub)
        assert call(*other) is False
        other[i] = args[i].cpu()
        assert call(*other) is False
        with pytest.raises(AssertionError):
            entry(*other)
    wrong = list(args)
    wrong[o] = args[o][..., :-1]                          # another shape, or not contiguous
    assert call(*wrong) is False
    with pytest.raises(AssertionError):
        entry(*wrong)
    with Watch():
        assert call(*args) is False
    taken = []
    with pytest.raises(Exception):                        # a wrapper has no memory of its own, before as now
        torch.vmap(lambda t: (taken.append(call(t, *args[1:])), entry(t, *args[1:]))[1])(args[0][None])
    assert taken == [False]
    assert call(*args[:-1]) is False
    torch.cuda.synchronize()
    assert not args[o].any(), "a call that was not taken wrote"


def test_tap_arrays_of_any_kind():
    import torch
    args, _ = usual(torch)["fir1d"]
    taps = args[2]
    fir = hb._calls.fir1d
    assert fir(args[0], args[1], taps.view(np.float16), 4) is True
    ref = args[1].clone()
    for other, took in ((taps.astype(">u2"), False), (np.repeat(taps, 2)[::2], False), (taps.reshape(3, 3), True), (list(map(int, taps)), False),
                        (taps.astype(np.int64), False)):
        args[1].zero_()
        assert fir(args[0], args[1], other, 4) is took
        hb.hb_fir1d(args[0], args[1], other, 4)
        assert torch.equal(ref, args[1])
    for anchor in (np.int64(4), 4.0, True):
        assert fir(args[0], args[1], taps, anchor) is False
    assert hb._calls.conv2d(args[0], args[1], taps, 0, 0) is False          # one dimension
    big = np.zeros(4096, dtype=np.uint16)
    for t, a in ((taps, 9), (taps, -1), (big, 0), (taps[:0], 0)):           # the library's own errors, by either way
        with pytest.raises(hb.HbError) as e:
            hb.hb_fir1d(args[0], args[1], t, a)
        assert e.value.code in (hb.HB_ERR_INVALID_ARG, hb.HB_ERR_UNSUPPORTED) and str(e.value).startswith("hb_fir1d failed: ")
