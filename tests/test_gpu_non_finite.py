"""How far a non-finite sample reaches.  The windows of the matrix formulation hold samples with zero weight, which make NaN
of an infinity: the header states how much further than the filter itself that may go."""
import numpy as np
import pytest

from paper_2512_02371_amd import synth

pytestmark = pytest.mark.gpu

H, W = 150, 333
PLACES = [(70, 160), (0, 0), (149, 332), (15, 31), (64, 128), (79, 207), (131, 4)]


def image(seed, *shape):
    import torch
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    return torch.randint(0, 2048, shape, generator=gen, device="cuda:0", dtype=torch.int16).float().div_(2048).half()


def check(call, y, x, value, own, more, shape=(H, W), scale=1.0):
    """Outputs further from the sample than `own` + `more` (up, down, left, right; in output samples) are those of the finite
    image, bit for bit; the ones that read the sample (`own`, when given) are not finite."""
    import torch
    img = image(5, H, W)
    clean = call(img)
    img[y, x] = value
    got = call(img)
    torch.cuda.synchronize()
    up, down, left, right = (o + m for o, m in zip(own, more))
    r, c = int(y * scale), int(x * scale)
    outside = np.ones(shape, dtype=bool)
    outside[max(0, r - up):r + down + 1, max(0, c - left):c + right + 1] = False
    a, b = clean.cpu().numpy(), got.cpu().numpy()
    changed = ~((a == b) | (np.isnan(a) & np.isnan(b)))
    where = np.argwhere(changed & outside)
    assert where.size == 0, f"({y}, {x}): outputs {where.min(0)} .. {where.max(0)} changed"
    assert not np.isfinite(b).all(), "the sample left no trace"


def out(*shape):
    import torch
    return torch.empty(shape, dtype=torch.float32, device="cuda:0")


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("y,x", PLACES)
def test_reach_of_a_non_finite_sample(y, x, value):
    from paper_2512_02371_amd import hb
    import torch
    for T, a in ((5, 2), (40, 7), (150, 149)):
        t = synth.random_taps_f16(T, T)
        # output x reads x - a .. x + T - 1 - a; clamping lets an edge sample reach no further than that
        check(lambda i: hb.hb_fir1d(i, out(H, W), t, a), y, x, value, (0, 0, T - 1 - a, a), (0, 0, 47, 47))
    for T, a in ((5, 2), (31, 15), (64, 3)):
        t = synth.gaussian_taps_f16(T, max(T / 5.0, 0.6))
        check(lambda i: hb.hb_sepblur(i, out(H, W), t, a, t, a), y, x, value, (T - 1 - a, a, T - 1 - a, a), (31, 31, 47, 47))
    for k, a in ((3, 1), (16, 0), (31, 30)):
        t = synth.random_kernel2d_f16(k, k, k)
        check(lambda i: hb.hb_conv2d(i, out(H, W), t, a, a), y, x, value, (k - 1 - a, a, k - 1 - a, a), (1, 1, 47, 47))
        check(lambda i: hb.hb_down2(i, out((H + 1) // 2, (W + 1) // 2), t, a, a), y, x, value, ((k - 1 - a) // 2 + 1, a // 2 + 1) * 2,
              (2, 2, 47, 47), ((H + 1) // 2, (W + 1) // 2), 0.5)
    for k, a in ((4, 0), (16, 7), (32, 2)):
        t = synth.random_kernel2d_f16(k, k, k)
        check(lambda i: hb.hb_up2(i, out(2 * H, 2 * W), t, a, a), y, x, value, (k - 2 * a, 2 * a + 1) * 2, (2, 2, 47, 47), (2 * H, 2 * W), 2.0)
    for part in (0, 1):
        def level(i):
            # an even width: the last column and row stay out
            i = i[:, :W - 1]
            r, d = out(H, W - 1), torch.empty((H // 2, (W - 1) // 2), dtype=torch.float16, device="cuda:0")
            hb.hb_pyr_level(i, r, d)
            return (r, d)[part]
        if x < W - 1:
            check(level, y, x, value, (6, 6, 6, 6) if part == 0 else (2, 2, 2, 2), (31, 31, 47, 47), ((H, W - 1), (H // 2, (W - 1) // 2))[part],
                  1.0 if part == 0 else 0.5)


@pytest.mark.parametrize("y,x", PLACES)
def test_reach_in_resize(y, x):
    """Outputs are taken in aligned groups of 16; a group's windows are widened by up to 48 samples along either axis."""
    from paper_2512_02371_amd import hb
    import torch
    for Ho, Wo in ((100, 200), (20, 30), (150, 333), (7, 17)):
        (sy, cy), (sx, cx) = hb.hb_lanczos3_matrix(H, Ho), hb.hb_lanczos3_matrix(W, Wo)
        dev = lambda a: torch.from_numpy(a).cuda()
        ws = torch.empty(hb.hb_resize_workspace_size(1, H, Wo), dtype=torch.uint8, device="cuda:0")

        def call(i):
            o = out(1, Ho, Wo)
            hb.hb_resize(i[None], o, ws, dev(sy), dev(cy.view(np.float16)), dev(sx), dev(cx.view(np.float16)))
            return o[0]
        grow = [int(np.ceil(n * (48 + 3 * m / n) / m)) + 16 for n, m in ((Ho, H), (Wo, W))]
        img = image(6, H, W)
        a = call(img).cpu().numpy()
        img[y, x] = float("inf")
        b = call(img).cpu().numpy()
        outside = np.ones((Ho, Wo), dtype=bool)
        r, c = y * Ho // H, x * Wo // W
        outside[max(0, r - grow[0]):r + grow[0] + 1, max(0, c - grow[1]):c + grow[1] + 1] = False
        assert np.array_equal(a[outside], b[outside]), f"{Ho}x{Wo} ({y}, {x})"


def test_reach_in_iir2_and_sat2d():
    """The recursion passes everything on; backwards a sample reaches its block of 32 (hb_iir2) or tile of 64 (hb_sat2d)."""
    from paper_2512_02371_amd import hb
    import torch
    sig = image(7, 2, 5000)
    ws = torch.empty(hb.hb_iir2_workspace_size(2, 5000), dtype=torch.uint8, device="cuda:0")
    for t in (0, 31, 32, 700, 4999):
        s = sig.clone()
        a = hb.hb_iir2(s, out(2, 5000), 1.2, -0.52, ws).cpu().numpy()
        s[1, t] = float("inf")
        b = hb.hb_iir2(s, out(2, 5000), 1.2, -0.52, ws).cpu().numpy()
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1, :t // 32 * 32], b[1, :t // 32 * 32]), t
        assert not np.isfinite(b[1, t])
    img = image(8, 200, 300)
    ws = torch.empty(hb.hb_sat2d_workspace_size(200, 300), dtype=torch.uint8, device="cuda:0")
    for y, x in ((0, 0), (63, 64), (100, 200), (199, 299)):
        i = img.clone()
        a = hb.hb_sat2d(i, out(200, 300), ws).cpu().numpy()
        i[y, x] = float("inf")
        b = hb.hb_sat2d(i, out(200, 300), ws).cpu().numpy()
        y0, x0 = y // 64 * 64, x // 64 * 64
        assert np.array_equal(a[:y0], b[:y0]) and np.array_equal(a[:, :x0], b[:, :x0]), (y, x)
        assert not np.isfinite(b[y, x])
