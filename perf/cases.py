"""The calls whose speed is tracked: every stage of the library through its Python entry points.

``listed()`` holds the sizes that the repository's benchmark and tests use, from one launch on a
small image to a whole 8192 x 8192 pyramid; ``draw()`` gives more calls of the same ranges.  Inputs
are drawn on the GPU from the seed with the distributions of ``paper_2512_02371_amd.synth`` (images
uniform on the fp16 grid of [0, 1), signals and conv activations uniform on the grid of [-1, 1)).
"""
from __future__ import annotations

import math

import torch

from paper_2512_02371_amd import hb, synth


def listed():
    return [
        # the smallest call of the benchmark: a short row filter on a small image (launch latency)
        {"name": "fir1d_256x256_t8", "op": "fir1d", "H": 256, "W": 256, "taps": 8, "pad": 0},
        # the large-tap study on a full image: a 256-tap row filter
        {"name": "fir1d_4096x4096_t256", "op": "fir1d", "H": 4096, "W": 4096, "taps": 256, "pad": 0},
        # the benchmark's Gaussian blur, 16 taps per axis
        {"name": "sepblur_4096x4096_t16", "op": "sepblur", "H": 4096, "W": 4096, "taps_x": 16, "taps_y": 16, "pad": 0},
        # a wider blur of a video-frame-sized image with odd sides (rows not dword aligned, ragged tiles)
        {"name": "sepblur_1079x1917_t31", "op": "sepblur", "H": 1079, "W": 1917, "taps_x": 31, "taps_y": 31, "pad": 0},
        # the benchmark's summed-area table
        {"name": "sat2d_4096x4096", "op": "sat2d", "H": 4096, "W": 4096, "pad": 0},
        # the benchmark's convolution layer (the one case bound by the matrix units)
        {"name": "conv3x3_1x1024x1024", "op": "conv3x3", "N": 1, "H": 1024, "W": 1024},
        # a Laplacian pyramid of the benchmark's image: each level reads the coarse image of the one before
        {"name": "pyramid_8192x8192_l3", "op": "pyramid", "H": 8192, "W": 8192, "levels": 3},
        # a dense, non-separable 2-D filter at the largest kernel size
        {"name": "conv2d_4096x4096_k32", "op": "conv2d", "H": 4096, "W": 4096, "kh": 32, "kw": 32, "pad": 0},
        # both directions of resampling by two between 4096^2 and 2048^2 (reduce one image, expand another)
        {"name": "resample2_4096x4096_k16", "op": "resample2", "H": 4096, "W": 4096, "k": 16, "pad": 0},
        # a thumbnail of a four-megapixel RGB image with the Lanczos filter
        {"name": "resize_3x2048x2048_450", "op": "resize", "C": 3, "H": 2048, "W": 2048, "Ho": 450, "Wo": 450},
        # a resonant filter over 50 s of stereo audio
        {"name": "iir2_2x2097152", "op": "iir2", "C": 2, "T": 1 << 21, "radius": 0.8944, "angle": 0.4636},
        # transform-domain denoising of a one-megapixel RGB image
        {"name": "dct_3x1024x1024", "op": "dct", "C": 3, "H": 1024, "W": 1024, "threshold": 0.25},
    ]


_OPS = ["fir1d", "sepblur", "sat2d", "conv3x3", "pyramid", "conv2d", "resample2", "resize", "iir2", "dct"]


def _log_int(rng, lo, hi):
    """An integer from lo to hi, spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _image(rng, lo, hi, most, step=1):
    """Height and width: a side from lo to hi, an aspect ratio from 1:4 to 4:1, at most `most` pixels; half of
    the images have sides that are multiples of 16, the others any multiple of `step`."""
    side = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    aspect = 2.0 ** rng.uniform(-1.0, 1.0)
    H, W = side * aspect, side / aspect
    shrink = min(1.0, math.sqrt(most / (H * W)))
    q = max(16, step) if rng.random() < 0.5 else step
    return tuple(max(q, int(v * shrink) // q * q) for v in (H, W))


def draw(rng):
    op = rng.choice(_OPS)
    pad = rng.choice([0, 0, 0, 64])          # a window of a wider image: its rows are `pad` pixels further apart
    if op == "fir1d":
        H, W = _image(rng, 64, 8192, 1 << 25)
        return {"op": op, "H": H, "W": W, "taps": _log_int(rng, 3, 256), "pad": pad}
    if op == "sepblur":
        H, W = _image(rng, 64, 8192, 1 << 25)
        t = _log_int(rng, 3, 64)
        return {"op": op, "H": H, "W": W, "taps_x": t, "taps_y": t if rng.random() < 0.7 else _log_int(rng, 3, 64), "pad": pad}
    if op == "sat2d":
        H, W = _image(rng, 64, 8192, 1 << 25)
        return {"op": op, "H": H, "W": W, "pad": pad}
    if op == "conv3x3":
        H, W = _image(rng, 14, 1024, 1 << 20)
        return {"op": op, "N": rng.randint(1, max(1, min(8, (1 << 20) // (H * W)))), "H": H, "W": W}
    if op == "pyramid":
        levels = rng.randint(1, 4)
        H, W = _image(rng, 128, 8192, 1 << 25, 1 << levels)
        return {"op": op, "H": H, "W": W, "levels": levels}
    if op == "conv2d":
        H, W = _image(rng, 64, 4096, 1 << 24)
        kh = _log_int(rng, 3, 32)
        return {"op": op, "H": H, "W": W, "kh": kh, "kw": kh if rng.random() < 0.7 else _log_int(rng, 3, 32), "pad": pad}
    if op == "resample2":
        H, W = _image(rng, 64, 4096, 1 << 24, 2)
        return {"op": op, "H": H, "W": W, "k": 2 * _log_int(rng, 2, 16), "pad": pad}
    if op == "resize":
        C = rng.choice([1, 3])
        H, W = _image(rng, 64, 4096, (1 << 24) // C)
        f = math.exp(rng.uniform(math.log(1.1), math.log(16.0)))
        return {"op": op, "C": C, "H": H, "W": W, "Ho": max(1, int(H / f)), "Wo": max(1, int(W / f))}
    if op == "iir2":
        C = _log_int(rng, 1, 64)
        return {"op": op, "C": C, "T": _log_int(rng, 1000, min(1 << 22, (1 << 23) // C)),
                "radius": round(rng.uniform(0.3, 0.95), 4), "angle": round(rng.uniform(0.1, 3.0), 4)}
    H, W = _image(rng, 64, 2048, 1 << 22, 8)
    C = rng.choice([1, 3])
    return {"op": op, "C": C, "H": H, "W": W, "threshold": round(rng.uniform(0.05, 0.5), 3)}


# ---- what a program holds before the call ---------------------------------------------------------------

def _uniform01(gen, *shape, pad=0):
    full = shape[:-1] + (shape[-1] + pad,)
    x = torch.randint(0, 2048, full, generator=gen, device="cuda", dtype=torch.int16).to(torch.float32).div_(2048.0).half()
    return x[..., :shape[-1]]


def _uniform_pm1(gen, *shape):
    return torch.randint(-1024, 1024, shape, generator=gen, device="cuda", dtype=torch.int16).to(torch.float32).div_(1024.0).half()


def _f32(*shape):
    return torch.empty(shape, dtype=torch.float32, device="cuda")


def _scratch(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device="cuda")


def _gaussian(taps):
    return synth.gaussian_taps_f16(taps, max(0.6, 3.0 * taps / 16.0))


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    op = case["op"]
    s = {"op": op}
    if op in ("fir1d", "sepblur", "conv2d", "sat2d"):
        H, W = case["H"], case["W"]
        s.update(x=_uniform01(gen, H, W, pad=case["pad"]), out=_f32(H, W))
        if op == "fir1d":
            s.update(taps=synth.random_taps_f16(seed, case["taps"]), anchor=(case["taps"] - 1) // 2)
        elif op == "sepblur":
            s.update(tx=_gaussian(case["taps_x"]), ty=_gaussian(case["taps_y"]),
                     ax=(case["taps_x"] - 1) // 2, ay=(case["taps_y"] - 1) // 2)
        elif op == "conv2d":
            s.update(taps=synth.random_kernel2d_f16(seed, case["kh"], case["kw"]),
                     ay=(case["kh"] - 1) // 2, ax=(case["kw"] - 1) // 2)
        else:
            s.update(ws=_scratch(hb.hb_sat2d_workspace_size(H, W)))
    elif op == "conv3x3":
        N, H, W = case["N"], case["H"], case["W"]
        w = torch.randn((3, 3, 64, 64), generator=gen, device="cuda").div_(24.0).half()
        s.update(x=_uniform_pm1(gen, N, H, W, 64), w=w, out=torch.empty((N, H, W, 64), dtype=torch.float16, device="cuda"))
    elif op == "pyramid":
        H, W, n = case["H"], case["W"], case["levels"]
        s.update(x=_uniform01(gen, H, W), residuals=[_f32(H >> i, W >> i) for i in range(n)],
                 coarse=[torch.empty((H >> i, W >> i), dtype=torch.float16, device="cuda") for i in range(1, n + 1)])
    elif op == "resample2":
        H, W, k = case["H"], case["W"], case["k"]
        s.update(x=_uniform01(gen, H, W, pad=case["pad"]), small=_uniform01(gen, H // 2, W // 2, pad=case["pad"]),
                 reduced=_f32(H // 2, W // 2), expanded=_f32(H, W), taps=synth.random_kernel2d_f16(seed, k, k),
                 down_anchor=(k - 1) // 2, up_anchor=(k // 2 - 1) // 2)
    elif op == "resize":
        C, H, W, Ho, Wo = (case[k] for k in ("C", "H", "W", "Ho", "Wo"))
        s.update(x=_uniform01(gen, C, H, W), out=_f32(C, Ho, Wo), ws=_scratch(hb.hb_resize_workspace_size(C, H, Wo)))
        for axis, n_in, n_out in (("y", H, Ho), ("x", W, Wo)):
            start, coef = hb.hb_lanczos3_matrix(n_in, n_out)
            s["start_" + axis] = torch.from_numpy(start).cuda()
            s["coef_" + axis] = torch.from_numpy(coef.view("float16")).cuda()
    elif op == "iir2":
        C, T = case["C"], case["T"]
        s.update(x=_uniform_pm1(gen, C, T), out=_f32(C, T), ws=_scratch(hb.hb_iir2_workspace_size(C, T)),
                 alpha=2.0 * case["radius"] * math.cos(case["angle"]), beta=-case["radius"] ** 2)
    else:
        C, H, W = case["C"], case["H"], case["W"]
        s.update(x=_uniform01(gen, C, H, W), out=_f32(C, H, W), ws=_scratch(hb.hb_dct_denoise_workspace_size(C, H, W)),
                 threshold=case["threshold"])
    return s


# ---- one pass -------------------------------------------------------------------------------------------

def _pyramid(s):
    x = s["x"]
    for residual, coarse in zip(s["residuals"], s["coarse"]):
        hb.hb_pyr_level(x, residual, coarse)
        x = coarse
    return s["residuals"] + s["coarse"]


def _resample2(s):
    return [hb.hb_down2(s["x"], s["reduced"], s["taps"], s["down_anchor"], s["down_anchor"]),
            hb.hb_up2(s["small"], s["expanded"], s["taps"], s["up_anchor"], s["up_anchor"])]


_RUN = {
    "fir1d": lambda s: hb.hb_fir1d(s["x"], s["out"], s["taps"], s["anchor"]),
    "sepblur": lambda s: hb.hb_sepblur(s["x"], s["out"], s["tx"], s["ax"], s["ty"], s["ay"]),
    "sat2d": lambda s: hb.hb_sat2d(s["x"], s["out"], s["ws"]),
    "conv3x3": lambda s: hb.hb_conv3x3(s["x"], s["w"], s["out"]),
    "pyramid": _pyramid,
    "conv2d": lambda s: hb.hb_conv2d(s["x"], s["out"], s["taps"], s["ay"], s["ax"]),
    "resample2": _resample2,
    "resize": lambda s: hb.hb_resize(s["x"], s["out"], s["ws"], s["start_y"], s["coef_y"], s["start_x"], s["coef_x"]),
    "iir2": lambda s: hb.hb_iir2(s["x"], s["out"], s["alpha"], s["beta"], s["ws"]),
    "dct": lambda s: hb.hb_dct_denoise(s["x"], s["out"], s["threshold"], s["ws"]),
}


def run(state):
    return _RUN[state["op"]](state)


# ---- what a pass cannot do without ----------------------------------------------------------------------

def work(case):
    """Input bytes once, output bytes once; the multiply-adds of each stage's definition, two flops each."""
    op = case["op"]
    if op == "conv3x3":
        px = case["N"] * case["H"] * case["W"]
        return {"bytes": 256 * px + 2 * 9 * 64 * 64, "flops": 2 * 9 * 64 * 64 * px}
    if op == "iir2":
        n = case["C"] * case["T"]
        return {"bytes": 6 * n, "flops": 4 * n}
    px = case["H"] * case["W"]
    if op == "fir1d":
        return {"bytes": 6 * px, "flops": 2 * case["taps"] * px}
    if op == "sepblur":
        return {"bytes": 6 * px, "flops": 2 * (case["taps_x"] + case["taps_y"]) * px}
    if op == "conv2d":
        return {"bytes": 6 * px, "flops": 2 * case["kh"] * case["kw"] * px}
    if op == "sat2d":
        return {"bytes": 6 * px, "flops": 2 * px}
    if op == "pyramid":
        total = sum(px >> (2 * i) for i in range(case["levels"]))
        return {"bytes": 6 * total + total // 2, "flops": 17 * total}
    if op == "resample2":
        return {"bytes": (2 * px + px) + (px // 2 + 4 * px), "flops": 2 * case["k"] ** 2 * (px // 4) * 2}
    if op == "resize":
        C, H, W, Ho, Wo = (case[k] for k in ("C", "H", "W", "Ho", "Wo"))
        bx, by = hb.hb_lanczos3_band(W, Wo), hb.hb_lanczos3_band(H, Ho)
        return {"bytes": 2 * C * px + 4 * C * Ho * Wo + 2 * (Wo * bx + Ho * by), "flops": 2 * C * (H * Wo * bx + Ho * Wo * by)}
    return {"bytes": 6 * case["C"] * px, "flops": case["C"] * (case["H"] // 8 - 1) * (case["W"] // 8 - 1) * 4 * 2 * 16 ** 3}


# About four times the distance measured between the stages and their definitions in fp64 (2-norm relative;
# "max" relative to the root mean square).
_TOLERANCE = {
    "fir1d": {"rel": 4e-7, "max": 2e-6},       # fp32 sums: 8e-8 / 4e-7 at 256 taps
    "conv2d": {"rel": 4e-7, "max": 2e-6},      # fp32 sums: 8e-8 / 4e-7 at 32 x 32
    "resample2": {"rel": 4e-7, "max": 2e-6},   # fp32 sums: 8e-8 / 4e-7
    "sat2d": {"rel": 4e-7, "max": 2e-6},       # fp32 sums over the image: 8e-8 / 5e-7
    "sepblur": {"rel": 6e-4, "max": 2e-3},     # fp16 intermediate: 1.5e-4 / 4.5e-4
    "conv3x3": {"rel": 8e-4, "max": 2e-3},     # fp16 results: 2.1e-4 / 4.9e-4
    "resize": {"rel": 7e-4, "max": 2.6e-3},    # fp16 intermediate: 1.8e-4 / 6.5e-4
    "iir2": {"rel": 2e-6, "max": 3.4e-5},      # fp32 sums through a resonant filter: 5.3e-7 / 8.4e-6
    # fp32 transforms: 1.4e-7 / 7.5e-6 where every bin falls on the same side of the threshold; a bin within
    # rounding of it may be kept by one implementation and cut by another, which moves its tile by up to
    # threshold / 8 (the transform's largest entry squared)
    "dct": {"rel": 1e-3, "max": 0.15},
}


def tolerance(case):
    if case["op"] == "pyramid":
        # fp16 intermediates against residuals that shrink from level to level as the image gets smoother:
        # 4.2e-4, 1.7e-3, 3.9e-3 and 8.0e-3 at levels one to four (max 1.9e-3, 7.1e-3, 1.4e-2 and 2.9e-2)
        return {"rel": (1.7e-3, 6.8e-3, 1.6e-2, 3e-2)[case["levels"] - 1],
                "max": (8e-3, 2.8e-2, 5.6e-2, 0.116)[case["levels"] - 1]}
    return _TOLERANCE[case["op"]]
