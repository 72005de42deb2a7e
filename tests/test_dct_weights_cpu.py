"""The windowed DCT matrix as the fp16 parts that hb_dct_denoise multiplies pixels with."""
import numpy as np


def windowed_dct():
    u, i = np.mgrid[0:16, 0:16].astype(np.float64)
    d = np.where(u == 0, 0.25, np.sqrt(2.0 / 16.0) * np.cos(np.pi * (2 * i + 1) * u / 32))
    return (d * np.sin(np.pi * (i + 0.5) / 16)).astype(np.float32)


def test_three_scaled_fp16_parts_are_the_fp32_weight():
    """hi + lo + rest of 1024 E, each rounded to fp16, is 1024 E itself: no weight is held in fewer bits than fp32, and
    the low parts are far from fp16's smallest numbers.  Two parts are not enough."""
    v = np.float32(1024) * windowed_dct()
    hi = v.astype(np.float16)
    lo = (v - hi.astype(np.float32)).astype(np.float16)
    rest = (v - hi.astype(np.float32) - lo.astype(np.float32)).astype(np.float16)
    exact = v.astype(np.float64)
    assert np.array_equal(hi.astype(np.float64) + lo.astype(np.float64) + rest.astype(np.float64), exact)
    assert not np.array_equal(hi.astype(np.float64) + lo.astype(np.float64), exact)
    assert np.all(np.isfinite(hi))


def test_the_kernel_s_tables_are_the_windowed_dct():
    """The tables in the source: E and its transpose to the last bit of fp32, the window."""
    import os
    import re
    src = open(os.path.join(os.path.dirname(__file__), "..", "paper_2512_02371_amd", "csrc", "dct.hip")).read()

    def table(name):
        body = re.search(name + r"\[\d+\] = \{([^}]*)\}", src).group(1)
        return np.array([float(v.rstrip("f")) for v in re.findall(r"[-+.\de]+f", body)], np.float64).astype(np.float32)

    e = windowed_dct()
    assert np.array_equal(table("kDctE").reshape(16, 16), e)
    assert np.array_equal(table("kDctEt").reshape(16, 16), e.T)
    assert np.array_equal(table("kDctW"), np.sin(np.pi * (np.arange(16) + 0.5) / 16).astype(np.float32))
