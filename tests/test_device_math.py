"""The sine and cosine polynomials of csrc/device_math.h against double precision, from the coefficients as the header holds
them (Cephes sinf / cosf).  No GPU is touched."""
import os
import re

import numpy as np

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2307_07649_amd", "csrc", "device_math.h")


def coefficients():
    text = open(HEADER).read()
    out = []
    for name in ("sp", "cp"):
        expr = re.search(r"const float %s = (.*?);" % name, text, flags=re.S).group(1)
        out.append([float(c) for c in re.findall(r"(-?\d\.\d+e-\d)f", expr)])
    return out


def polynomials(x, sin_c, cos_c):
    t = x.dtype.type
    s, c = [t(v) for v in sin_c], [t(v) for v in cos_c]
    x2 = x * x
    return (x + x * x2 * (s[0] + x2 * (s[1] + x2 * s[2])),
            t(1) - t(0.5) * x2 + x2 * x2 * (c[0] + x2 * (c[1] + x2 * c[2])))


def test_sine_and_cosine_polynomials():
    sin_c, cos_c = coefficients()
    assert len(sin_c) == 3 and len(cos_c) == 3
    x = np.linspace(-np.pi / 4, np.pi / 4, 1_000_001)
    s, c = polynomials(x, sin_c, cos_c)
    assert np.abs(s - np.sin(x)).max() <= 2.7e-9 and np.abs(c - np.cos(x)).max() <= 1.1e-10
    # in float, with half an ulp of numbers in [0.5, 1) being 3.0e-8.  Cosine: the result and 1 - x^2 / 2 are rounded, and
    # x^2 at half its weight: 7.5e-8.  Sine: the result is rounded, x^2 at a weight of x / 6, and the correction (at most
    # 0.081) and its last factor by 3.7e-9 each, beside the polynomial's own 2.7e-9: 4.6e-8
    x = x.astype(np.float32)
    s, c = polynomials(x, sin_c, cos_c)
    assert np.abs(s - np.sin(x.astype(np.float64))).max() <= 4.6e-8
    assert np.abs(c - np.cos(x.astype(np.float64))).max() <= 7.5e-8
