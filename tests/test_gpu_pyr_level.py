"""hb_pyr_level / hb_pyr_level_valu against the fp64 oracle, element by element."""
import numpy as np
import pytest

from paper_2512_02371_amd import synth
from hbtest import assert_close, padded, up

pytestmark = pytest.mark.gpu

CASES = [(64, 64), (2, 2), (4, 6), (34, 70), (130, 300), (256, 256), (96, 62), (66, 192), (30, 1026)]


def run(fn, H, W, want_down, pitch_extra=0, seed=0):
    import torch
    from paper_2512_02371_amd import hb
    img = synth.uniform01_f16(5000 + seed + H * 3 + W, (H, W))
    d_in = up(img)
    if pitch_extra:
        _, d_in = padded(d_in, W + pitch_extra)
    rbuf, res = padded(torch.zeros((H, W), dtype=torch.float32, device="cuda:0"), W + pitch_extra)
    dbuf, down = padded(torch.zeros((H // 2, W // 2), dtype=torch.float16, device="cuda:0"), W // 2 + pitch_extra)
    print(f"{fn} H={H} W={W} down={want_down} pitch+{pitch_extra}", flush=True)
    getattr(hb, fn)(d_in, res, down if want_down else None)
    torch.cuda.synchronize()
    return img, res.cpu().numpy(), down.cpu().numpy(), rbuf.cpu().numpy(), dbuf.cpu().numpy()


@pytest.mark.parametrize("fn", ["hb_pyr_level", "hb_pyr_level_valu"])
@pytest.mark.parametrize("H,W", CASES)
def test_pyr_matches_oracle(orc, fn, H, W):
    img, res, down, _, _ = run(fn, H, W, True)
    ref, dref = orc.pyr_level(img, want_down=True)
    assert_close(res, ref, f"{fn} residual {H}x{W}")
    assert_close(down.astype(np.float64), dref, f"{fn} down {H}x{W}")


@pytest.mark.parametrize("fn", ["hb_pyr_level", "hb_pyr_level_valu"])
def test_pyr_without_down_and_with_pitch(orc, fn):
    H, W = 70, 150
    img, res, down, rbuf, dbuf = run(fn, H, W, False, pitch_extra=6)
    assert_close(res, orc.pyr_level(img), f"{fn} pitched")
    assert np.all(rbuf[:, W:] == 7.0) and np.all(dbuf == np.float16(7.0)) or np.all(down == 0), "stray writes"
    assert np.all(down == 0), "down written although not requested"


@pytest.mark.parametrize("pitch_extra", [5, 8])
def test_pyr_pitched_image_with_interior_tasks(orc, pitch_extra):
    """Large enough for interior tasks; an odd pitch puts every second row on a 2-byte boundary."""
    H, W = 130, 300
    img, res, down, rbuf, dbuf = run("hb_pyr_level", H, W, True, pitch_extra=pitch_extra, seed=3)
    ref, dref = orc.pyr_level(img, want_down=True)
    assert_close(res, ref, f"pitched +{pitch_extra} residual")
    assert_close(down.astype(np.float64), dref, f"pitched +{pitch_extra} down")
    assert np.all(rbuf[:, W:] == 7.0), "stray writes beyond the row"


@pytest.mark.parametrize("fn", ["hb_pyr_level", "hb_pyr_level_valu"])
def test_pyr_constant_image_has_zero_residual(fn):
    import torch
    from paper_2512_02371_amd import hb
    H, W = 96, 160
    res = torch.ones((H, W), dtype=torch.float32, device="cuda:0")
    getattr(hb, fn)(up(synth.f64_to_f16_bits(np.full((H, W), 0.75))), res, None)
    assert float(res.abs().max()) == 0.0


@pytest.mark.parametrize("fn", ["hb_pyr_level", "hb_pyr_level_valu"])
def test_pyr_benchmark_width_slab(orc, fn):
    """A 320-row slab at the benchmark's 8192-pixel width: same strips as the full image."""
    import torch
    from paper_2512_02371_amd import hb
    H, W = 320, 8192
    img = synth.uniform01_f16(1005, (H, W))
    res = torch.zeros((H, W), dtype=torch.float32, device="cuda:0")
    getattr(hb, fn)(up(img), res, None)
    torch.cuda.synchronize()
    assert_close(res.cpu().numpy(), orc.pyr_level(img), fn)


@pytest.mark.parametrize("H,W", [(8, 8), (8, 74), (10, 40), (72, 8), (14, 18), (16, 104), (36, 36), (66, 74), (34, 2056), (1030, 46)])
def test_pyr_border_rows_and_columns_of_the_composite_matrix(orc, H, W):
    """Sizes around the ends of the 32 x 32 and 32 x 64 tasks and of the windows (8 pixels before a tile, 8 after),
    down to the smallest image whose two borders do not meet; tolerance as everywhere: one fp16 rounding of the
    row-filtered pixels, at most 2^-12 of a value below 1."""
    _, res, down, _, _ = out = run("hb_pyr_level", H, W, True, pitch_extra=3)
    ref, dref = orc.pyr_level(out[0], want_down=True)
    assert_close(res, ref, f"residual {H}x{W}")
    assert_close(down.astype(np.float64), dref, f"down {H}x{W}")


@pytest.mark.parametrize("want_down", [False, True])
def test_pyr_full_benchmark_size_sampled_bands(orc, want_down):
    """The benchmark's 8192 x 8192 launch (long interior tasks, many rounds of the tile ring), checked on
    row bands: the oracle runs on a crop with 16 rows of margin, whose inner rows do not see the crop."""
    import torch
    from paper_2512_02371_amd import hb
    H = W = 8192
    img = synth.uniform01_f16(1005, (H, W))
    res = torch.zeros((H, W), dtype=torch.float32, device="cuda:0")
    down = torch.zeros((H // 2, W // 2), dtype=torch.float16, device="cuda:0") if want_down else None
    print(f"hb_pyr_level {H}x{W} down={want_down}", flush=True)
    hb.hb_pyr_level(up(img), res, down)
    torch.cuda.synchronize()
    for y0 in (0, 16, 480, 1008, 2040, 4096 - 32, 6000, H - 96, H - 64):
        lo, hi = max(y0 - 16, 0), min(y0 + 64 + 16, H)
        ref, dref = orc.pyr_level(img[lo:hi], want_down=True)
        a, b = (0 if lo == 0 else 16), (hi - lo if hi == H else hi - lo - 16)
        assert_close(res[lo + a:lo + b].cpu().numpy(), ref[a:b], f"residual rows {lo + a}..{lo + b}")
        if want_down:
            got = down[(lo + a) // 2:(lo + b) // 2].cpu().numpy().astype(np.float64)
            assert_close(got, dref[a // 2:b // 2], f"down rows {(lo + a) // 2}..{(lo + b) // 2}")


def _up(d):
    """U of the definition, in float64, from a coarser level d."""
    def axis0(d):
        e = np.concatenate([d[:1], d, d[-1:]])
        u = np.empty((2 * d.shape[0], d.shape[1]))
        u[0::2] = (e[:-2] + 6 * e[1:-1] + e[2:]) / 8
        u[1::2] = (e[1:-1] + e[2:]) / 2
        return u
    return axis0(axis0(d.T).T)


def _down_axis0(p):
    e = np.concatenate([p[:1], p[:1], p, p[-1:], p[-1:]])
    n = p.shape[0] // 2
    return sum(w * e[i:i + 2 * n:2] for i, w in enumerate((0.0625, 0.25, 0.375, 0.25, 0.0625)))


ROUND_TRIP_SIZES = [(2, 48), (6, 50), (64, 64), (34, 70), (130, 300), (96, 104), (66, 202), (30, 1026), (1030, 88)]


@pytest.mark.parametrize("smooth", [False, True])
@pytest.mark.parametrize("fn", ["hb_pyr_level", "hb_pyr_level_valu"])
@pytest.mark.parametrize("H,W", ROUND_TRIP_SIZES + [(16, 46), (20, 8)])
def test_pyr_residual_belongs_to_the_coarser_level(fn, H, W, smooth):
    """residual + up(down) is the input: up to fp32 sums (three of numbers below 1: 3 * 2^-23) for the twin and for
    narrow images, up to the rounding of U along x otherwise (below 1: half of 2^-11, passed on with weights that add up
    to 1)."""
    import torch
    from paper_2512_02371_amd import hb
    img = synth.uniform01_f16(5800 + H + W, (H, W)).view(np.float16)
    if smooth:
        y, x = np.mgrid[0:H, 0:W]
        img = (0.5 + 0.45 * np.sin(y / 9.0) * np.cos(x / 13.0)).astype(np.float16)
    d_in = torch.from_numpy(img).to("cuda:0")
    res = torch.empty((H, W), dtype=torch.float32, device="cuda:0")
    down = torch.empty((H // 2, W // 2), dtype=torch.float16, device="cuda:0")
    getattr(hb, fn)(d_in, res, down)
    back = res.cpu().numpy().astype(np.float64) + _up(down.cpu().numpy().astype(np.float64))
    bound = 3 * 2.0 ** -23 + (2.0 ** -12 if fn == "hb_pyr_level" and W >= 48 else 0.0)
    assert np.abs(back - img.astype(np.float64)).max() <= bound


@pytest.mark.parametrize("H,W", ROUND_TRIP_SIZES)
def test_pyr_rounds_where_the_definition_of_the_stage_says(H, W):
    """The row-filtered pixels, D and U along x are fp16, every sum is fp32.  On the 2^-11 grid the sums are exact, so
    the roundings alone decide the results."""
    _, res, down, _, _ = out = run("hb_pyr_level", H, W, True)
    img = out[0].view(np.float16).astype(np.float64)
    f16 = lambda a: a.astype(np.float16).astype(np.float64)
    d = f16(_down_axis0(f16(_down_axis0(img.T).T)))
    e = np.concatenate([d[:, :1], d, d[:, -1:]], axis=1)
    u1 = np.empty((H // 2, W))
    u1[:, 0::2], u1[:, 1::2] = (e[:, :-2] + 6 * e[:, 1:-1] + e[:, 2:]) / 8, (e[:, 1:-1] + e[:, 2:]) / 2
    u1 = f16(u1)
    e = np.concatenate([u1[:1], u1, u1[-1:]])
    u = np.empty((H, W))
    u[0::2], u[1::2] = (e[:-2] + 6 * e[1:-1] + e[2:]) / 8, (e[1:-1] + e[2:]) / 2
    assert np.array_equal(down.astype(np.float64), d)
    assert np.abs(res - (img - u)).max() <= 2.0 ** -23
