"""The GELU of 16-bit models against the normal distribution function, on the
host: the device function's coefficients are read from its source and evaluated
in float32 in its order (division for the hardware reciprocal and exp2 for the
hardware exponential, each within 1 ulp).
"""
import os
import re

import numpy as np
from scipy.special import erfc

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2509_16248_amd", "csrc", "gm_gemm_epilogue.h")


def _device_gelu():
    body = open(SRC).read().split("float gelu_f(float x)", 1)[1].split("\n}\n", 1)[0]
    body = body.split("} else {", 1)[1]
    num = r"(-?[0-9.]+)f"
    slope, = re.findall(r"rcpf\(fmaf\(%s, ax, 1\.0f\)\)" % num, body)
    rate, = re.findall(r"exp2f\(ax \* ax \* %s\)" % num, body)
    poly = re.findall(r"float q = %s;" % num, body) + re.findall(r"q = fmaf\(q, t, %s\);" % num, body)
    assert len(poly) == 8
    f = np.float32
    # a fused multiply-add: the product of two float32 is exact in float64
    fma = lambda a, b, c: f(np.asarray(a, np.float64) * np.float64(b) + np.float64(c))

    def gelu(x):
        ax = np.abs(x)
        t = f(1) / fma(f(slope), ax, f(1))
        e = np.exp2(f(f(ax * ax) * f(rate)))
        q = f(poly[0])
        for c in poly[1:]:
            q = fma(q, t, f(c))
        h = f(f(q * t) * e)
        return f(x * np.where(x < 0, h, f(1) - h))
    return gelu


def test_relative_error():
    """The fit is within 1.5e-7, and each of the ~12 roundings adds at most
    6e-8: 1e-6 near zero.  Further out the exponent x^2 / 2 log2(e) itself is
    rounded twice, which moves exp2 by up to 2 x 6e-8 x x^2 / 2 more."""
    x = np.concatenate([np.linspace(-12, 12, 400001), np.geomspace(1e-6, 1, 1000)]).astype(np.float32)
    x = x[x != 0]
    x64 = x.astype(np.float64)
    exact = x64 * 0.5 * erfc(-x64 / np.sqrt(2))
    rel = np.abs(_device_gelu()(x) - exact) / np.abs(exact)
    assert rel[np.abs(x) < 1].max() < 1e-6
    assert (rel <= 1e-6 + 6e-8 * x64 * x64)[x > -12].all()


def test_tails():
    g = _device_gelu()
    big = np.float32(30000.0)
    assert g(big) == big and g(-big) == 0 and g(np.float32(0)) == 0
    assert np.isnan(g(np.float32(np.nan)))
