"""hb_resize / hb_resize_valu (resampling with banded matrices, Sec. V-C) against the fp64 oracle.
Both sides apply the SAME fp16 matrices (built by hb_lanczos3_matrix or drawn at random)."""
import numpy as np
import pytest

from paper_2512_02371_amd import synth
from hbtest import assert_close, up

pytestmark = pytest.mark.gpu


def run(fn, img, sy, cy, sx, cx, pitch_extra=0):
    """img: [C, H, W] fp16 bits; matrices as host arrays.  Returns the [C, Ho, Wo] result and its canary columns."""
    import torch
    from paper_2512_02371_amd import hb
    C, H, W = img.shape
    Ho, Wo = cy.shape[0], cx.shape[0]
    d_in = up(img)
    if pitch_extra:
        base = torch.full((C, H + 1, W + pitch_extra), 3.0, dtype=torch.float16, device="cuda:0")
        base[:, :H, :W] = d_in
        d_in = base[:, :H, :W]
    obuf = torch.full((C, Ho + 1, Wo + pitch_extra), 7.0, dtype=torch.float32, device="cuda:0")
    out = obuf[:, :Ho, :Wo]
    ws = torch.empty(hb.hb_resize_workspace_size(C, H, Wo), dtype=torch.uint8, device="cuda:0")
    dev = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0").view(t) if t else torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    d_sy, d_sx = dev(sy.astype(np.int32), None), dev(sx.astype(np.int32), None)
    d_cy, d_cx = dev(cy.view(np.int16), torch.float16), dev(cx.view(np.int16), torch.float16)
    print(f"{fn} C={C} {H}x{W} -> {Ho}x{Wo} bands {cy.shape[1]},{cx.shape[1]} pitch+{pitch_extra}", flush=True)
    getattr(hb, fn)(d_in, out, ws, d_sy, d_cy, d_sx, d_cx)
    torch.cuda.synchronize()
    return out.cpu().numpy(), obuf.cpu().numpy()


def lanczos(hb, n_in, n_out):
    return hb.hb_lanczos3_matrix(n_in, n_out)


@pytest.mark.parametrize("fn", ["hb_resize", "hb_resize_valu"])
@pytest.mark.parametrize("C,H,W,Ho,Wo", [
    (3, 256, 256, 115, 115),      # the paper's factors 2.22 .. 14.3 on a smaller image
    (3, 256, 320, 56, 70),
    (1, 300, 200, 31, 18),        # factor ~10: bands of 59 and 67 samples, groups span > 200 samples
    (2, 130, 190, 130, 190),      # same size: the identity matrix with its 7-sample band
    (1, 97, 131, 45, 100),        # ragged everything
    (3, 64, 64, 1, 1),            # one output sample
    (2, 254, 175, 3, 154),        # factor 85: band 509, the three rows together span 679 samples (two rounds)
    (1, 40, 1300, 30, 16),        # factor 81 along x: one group of 16 outputs spans the whole row (three rounds)
    (1, 1, 1, 1, 1),
])
def test_resize_lanczos_matches_oracle(orc, fn, C, H, W, Ho, Wo):
    from paper_2512_02371_amd import hb
    img = synth.uniform01_f16(9000 + H + 3 * W, (C, H, W))
    sy, cy = lanczos(hb, H, Ho)
    sx, cx = lanczos(hb, W, Wo)
    got, _ = run(fn, img, sy, cy, sx, cx)
    for c in range(C):
        assert_close(got[c], orc.band_resize(img[c], sy, cy, sx, cx), f"{fn} plane {c} {H}x{W}->{Ho}x{Wo}")


@pytest.mark.parametrize("fn", ["hb_resize", "hb_resize_valu"])
def test_resize_random_bands_and_irregular_starts(orc, fn):
    """Not a Lanczos matrix: random coefficients, starts that jump, repeat and leave the image on both sides."""
    C, H, W, Ho, Wo, by, bx = 2, 150, 210, 70, 90, 9, 14
    img = synth.uniform01_f16(9100, (C, H, W))
    cy = synth.random_kernel2d_f16(9101, Ho, by) .view(np.uint16)
    cx = synth.random_kernel2d_f16(9102, Wo, bx).view(np.uint16)
    # scale the rows back up (the generator normalises the whole array to sum |k| = 1)
    cy = (cy.view(np.float16).astype(np.float64) * Ho).astype(np.float16).view(np.uint16)
    cx = (cx.view(np.float16).astype(np.float64) * Wo).astype(np.float16).view(np.uint16)
    h = synth.hash_u64(9103, 0, Ho + Wo)
    sy = (np.arange(Ho) * 2 + (h[:Ho] % np.uint64(13)).astype(np.int64) - 8).astype(np.int32)
    sx = (np.arange(Wo) * 2 + (h[Ho:] % np.uint64(40)).astype(np.int64) - 15).astype(np.int32)
    sy[-1], sx[-1] = H + 5, W - 3                      # entirely / partly past the far edge
    got, _ = run(fn, img, sy, cy, sx, cx)
    for c in range(C):
        assert_close(got[c], orc.band_resize(img[c], sy, cy, sx, cx), f"{fn} plane {c}")


@pytest.mark.parametrize("fn", ["hb_resize", "hb_resize_valu"])
def test_resize_starts_far_apart_and_far_outside(orc, fn):
    """Starts of one group scattered over a long row (several rounds of the coefficient block) and
    starts far outside the image on both sides (every sample clamps to the first / last pixel)."""
    C, H, W, Ho, Wo, by, bx = 1, 70, 3000, 20, 40, 5, 33
    img = synth.uniform01_f16(9400, (C, H, W))
    cy = (synth.random_kernel2d_f16(9401, Ho, by).view(np.float16).astype(np.float64) * Ho).astype(np.float16).view(np.uint16)
    cx = (synth.random_kernel2d_f16(9402, Wo, bx).view(np.float16).astype(np.float64) * Wo).astype(np.float16).view(np.uint16)
    h = synth.hash_u64(9403, 0, Ho + Wo)
    sy = ((h[:Ho] % np.uint64(H + 20)).astype(np.int64) - 10).astype(np.int32)
    sx = ((h[Ho:] % np.uint64(W + 100)).astype(np.int64) - 50).astype(np.int32)
    sx[0], sx[1], sx[17], sx[18] = -(1 << 30), 1 << 30, -5000, 7000
    sy[0], sy[1] = -(2 ** 31), 2 ** 31 - 1
    got, _ = run(fn, img, sy, cy, sx, cx)
    assert_close(got[0], orc.band_resize(img[0], sy, cy, sx, cx), fn)


@pytest.mark.parametrize("C,H,W,Ho,Wo,by,bx,reach", [
    (1, 40, 7, 33, 40, 5, 3, 30),            # narrower than eight pixels
    (1, 900, 8, 40, 20, 400, 2, 900),        # fewer than eight samples of a row; rows in several rounds
    (2, 260, 1200, 17, 33, 3, 500, 700),     # spans of more than 384 columns
    (1, 300, 500, 135, 2090, 9, 12, 250),    # one group of rows per wave, rows in several rounds
    (1, 150, 900, 131, 8330, 20, 7, 60),     # two
    (1, 250, 700, 230, 9610, 30, 8, 20),     # four
])
def test_resize_random_starts_over_the_work_splits(orc, C, H, W, Ho, Wo, by, bx, reach):
    """Starts scattered around a ramp, some outside the image, over the sizes where the split of the work changes."""
    img = synth.uniform01_f16(9500 + H, (C, H, W))
    def matrix(seed, n, band, n_in):
        k = (synth.random_kernel2d_f16(seed, n, band).view(np.float16).astype(np.float64) * n).astype(np.float16).view(np.uint16)
        h = synth.hash_u64(seed + 1, 0, n)
        return (np.arange(n) * n_in // n + (h % np.uint64(reach)).astype(np.int64) - reach // 2).astype(np.int32), k
    sy, cy = matrix(9510 + Ho, Ho, by, H)
    sx, cx = matrix(9520 + Wo, Wo, bx, W)
    got, obuf = run("hb_resize", img, sy, cy, sx, cx, pitch_extra=3)
    for c in range(C):
        assert_close(got[c], orc.band_resize(img[c], sy, cy, sx, cx), f"plane {c}")
    assert np.all(obuf[:, :, Wo:] == 7.0) and np.all(obuf[:, Ho:, :] == 7.0), "wrote outside the output planes"


@pytest.mark.parametrize("C,H,W,Ho,Wo", [
    (1, 700, 900, 10, 13),        # two launches: spans of several hundred samples in both directions, a short last group
    (2, 131, 1029, 2, 17),        # ... a single row beyond two groups of 64, odd pitch
    (1, 4200, 500, 50, 20),       # ... factor 84
    (1, 3, 3000, 3, 60),          # ... few rows: one launch, more than 384 columns
    (3, 20, 2500, 18, 40),
    (400, 200, 40, 10, 40),       # waves that share a group of rows too long for one wave: 1200 groups
    (700, 200, 40, 10, 40),       # 2100, one to a column: two launches
    (1100, 200, 130, 10, 32),     # ... narrow results: one launch, shared all the same
    (240, 560, 48, 34, 40),       # three to a column: a wave each, in rounds
    (1, 770, 130, 22, 60),        # rows that start on odd samples and a group that spans many of them
])
def test_resize_large_factors(orc, C, H, W, Ho, Wo):
    """The routes of the large factors: Lanczos matrices, whose starts advance by the scale."""
    from paper_2512_02371_amd import hb
    img = synth.uniform01_f16(9600 + H + W, (C, H, W))
    sy, cy = lanczos(hb, H, Ho)
    sx, cx = lanczos(hb, W, Wo)
    got, obuf = run("hb_resize", img, sy, cy, sx, cx, pitch_extra=1)
    for c in sorted({0, C // 2, C - 1}):
        assert_close(got[c], orc.band_resize(img[c], sy, cy, sx, cx), f"plane {c}")
    assert np.all(obuf[:, :, Wo:] == 7.0) and np.all(obuf[:, Ho:, :] == 7.0), "wrote outside the output planes"


def test_resize_large_enlargement(orc):
    """Outputs of more than 64 MB with rows on line boundaries: two launches."""
    H, W, Ho, Wo = 40, 2060, 4097, 4128
    img = synth.uniform01_f16(9650, (1, H, W))
    rows = lambda seed, n: (synth.random_kernel2d_f16(seed, n, 3).view(np.float16).astype(np.float64) * n).astype(np.float16).view(np.uint16)
    sy, cy = (np.arange(Ho) * H // Ho).astype(np.int32) - 1, rows(9651, Ho)
    sx, cx = (np.arange(Wo) * W // Wo).astype(np.int32) - 1, rows(9652, Wo)
    got, obuf = run("hb_resize", img, sy, cy, sx, cx, pitch_extra=32)
    assert_close(got[0], orc.band_resize(img[0], sy, cy, sx, cx), "enlargement")
    assert np.all(obuf[:, :, Wo:] == 7.0) and np.all(obuf[:, Ho:, :] == 7.0), "wrote outside the output planes"


@pytest.mark.parametrize("fn", ["hb_resize", "hb_resize_valu"])
def test_resize_pitched_planes(orc, fn):
    from paper_2512_02371_amd import hb
    C, H, W, Ho, Wo = 2, 140, 203, 50, 77
    img = synth.uniform01_f16(9200, (C, H, W))
    sy, cy = lanczos(hb, H, Ho)
    sx, cx = lanczos(hb, W, Wo)
    got, obuf = run(fn, img, sy, cy, sx, cx, pitch_extra=5)
    for c in range(C):
        assert_close(got[c], orc.band_resize(img[c], sy, cy, sx, cx), f"{fn} plane {c}")
    assert np.all(obuf[:, :, Wo:] == 7.0) and np.all(obuf[:, Ho:, :] == 7.0), "wrote outside the output planes"


def test_resize_full_size(orc):
    """The paper's workload: a 2048 x 2048 RGB image to 143, 245, 450 and 921 squared; one plane each is
    compared in full (the oracle needs ~1 s per plane at the largest size)."""
    from paper_2512_02371_amd import hb
    C, H, W = 3, 2048, 2048
    img = synth.uniform01_f16(9300, (C, H, W))
    for n, c in ((143, 0), (245, 1), (450, 2), (921, 0)):
        s, k = lanczos(hb, H, n)
        got, _ = run("hb_resize", img, s, k, s, k)
        assert_close(got[c], orc.band_resize(img[c], s, k, s, k), f"2048 -> {n}, plane {c}")


@pytest.mark.parametrize("band", [2, 26, 28, 34])     # spans of 32 to 64 samples: at, just under and over whole chunks
@pytest.mark.parametrize("pitch_extra", [0, 1, 2])    # rows on 16 bytes, on every byte pair, on 4 bytes
def test_resize_first_column_of_a_window(orc, band, pitch_extra):
    """Windows that start on every residue of eight samples, inside the image and left of it."""
    H, W, Ho, Wo = 40, 72, 18, 20
    img = synth.uniform01_f16(9200 + band, (2, H, W))
    cx = (synth.random_kernel2d_f16(9201, Wo, band).view(np.float16).astype(np.float64) * Wo).astype(np.float16).view(np.uint16)
    from paper_2512_02371_amd import hb
    sy, cy = lanczos(hb, H, Ho)
    for off in range(-9, 9):
        sx = (off + 2 * np.arange(Wo)).astype(np.int32)
        got, _ = run("hb_resize", img, sy, cy, sx, cx, pitch_extra)
        for c in range(2):
            assert_close(got[c], orc.band_resize(img[c], sy, cy, sx, cx), f"offset {off} plane {c}")


# calls of odd pitches, by what the library makes of them (tests/test_resize_route_cpu.py holds it to that)
APART_SHARED = [                              # the waves of a workgroup share a group
    (3, 700, 1003, 97, 700), (1, 1100, 1555, 400, 601), (1, 1400, 2001, 300, 444),               # windows of one to four chunks
    (1, 1001, 3301, 181, 600), (1, 1600, 4601, 150, 307), (2, 1400, 2401, 100, 160),             # of more
    (1, 190, 40001, 17, 5000), (1, 2500, 2601, 125, 700),                                        # few groups of rows; more rows than a wave's own T holds
]
APART_OWN = [                                 # a group, two or four per wave
    (1, 300, 1201, 290, 1190), (2, 801, 1601, 700, 1400), (1, 2301, 2001, 2100, 1900),           # one chunk
    (1, 1800, 2801, 1200, 700), (2, 900, 3001, 600, 560), (3, 800, 3201, 700, 400), (2, 1601, 1801, 1400, 700),    # three, four, six, two
    (8, 1265, 2865, 221, 501),
]
NOT_APART = [(5, 500, 2101, 52, 1900), (8, 700, 2101, 73, 1900), (16, 300, 89, 180, 60), (1, 2701, 2601, 40, 40)]     # long groups in one launch and in two, narrow, a wide span


@pytest.mark.parametrize("first", [0, 1])             # the image's first row starts on an even or an odd sample
@pytest.mark.parametrize("C,H,W,Ho,Wo", APART_SHARED + APART_OWN + NOT_APART)
def test_resize_even_and_odd_rows_apart(orc, C, H, W, Ho, Wo, first):
    """Odd pitches: rows that start on even and on odd samples are read apart, or not."""
    import torch
    from paper_2512_02371_amd import hb
    (sy, cy), (sx, cx) = lanczos(hb, H, Ho), lanczos(hb, W, Wo)
    img = synth.uniform01_f16(3000 + H + first, (C, H, W))
    base = torch.full((C, H, W + 1 + W % 2), float("nan"), dtype=torch.float16, device="cuda:0")      # an odd pitch
    d_in = base[:, :, first:first + W]
    d_in.copy_(up(img))
    assert d_in.stride(1) % 2 == 1
    out = torch.full((C, Ho, Wo), 7.0, dtype=torch.float32, device="cuda:0")
    ws = torch.empty(hb.hb_resize_workspace_size(C, H, Wo), dtype=torch.uint8, device="cuda:0")
    dev = lambda a: torch.from_numpy(a).to("cuda:0")
    print(f"hb_resize C={C} {H}x{W} -> {Ho}x{Wo} first {first}", flush=True)
    hb.hb_resize(d_in, out, ws, dev(sy), dev(cy.view(np.float16)), dev(sx), dev(cx.view(np.float16)))
    torch.cuda.synchronize()
    for ch in range(C):
        assert_close(out[ch].cpu().numpy(), orc.band_resize(img[ch], sy, cy, sx, cx), f"hb_resize {H}x{W} -> {Ho}x{Wo} plane {ch}")
