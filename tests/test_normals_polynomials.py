"""The polynomials of the FP64 normals (cmflb_device.h: minus_two_log, turn)
against the functions they stand for, in extended precision over their whole
range: the fit errors that the source states.  CPU only; the rounding of the
device code around them is measured in test_gpu_normals_fp64.py."""
import os
import re

import numpy as np
import pytest

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                      "paper_2602_16486_amd", "csrc", "cmflb_device.h")
LD = np.longdouble


def constants(function):
    with open(HEADER) as fh:
        body = re.search(r"__device__ __forceinline__ \w+ " + function + r"\(.*?\n}\n", fh.read(), re.S).group()
    return [LD(float.fromhex(h)) for h in re.findall(r"-?0x1\.[0-9a-f]+p[+-]?\d+", body)]


def horner(coefs, x):
    p = np.zeros_like(x)
    for c in coefs:
        p = p * x + c
    return p


@pytest.fixture(autouse=True)
def _extended_precision():
    if np.finfo(LD).nmant < 63:
        pytest.skip("long double is no wider than double")


def test_logarithm():
    """-2 ln f = q + q R(q^2), f in [sqrt(1/2), sqrt(2)), q = -4 (f - 1) / (f + 1),
    R = z p(z): 5e-18 (as printed, to half a digit), and -2 ln 2 in two parts."""
    c = constants("minus_two_log")
    assert float(c[0]) == np.sqrt(0.5) and len(c) == 10
    # both ends and every second FP64 exponent towards f = 1
    q = LD(4) * (1 - np.sqrt(LD(0.5))) / (1 + np.sqrt(LD(0.5))) * np.concatenate(
        [np.linspace(LD(1), LD(1e-3), 200_001), LD(2) ** -np.arange(10, 26, 2)])
    t = q / 4  # -2 ln f = 4 atanh(t): the series, whose terms are all positive
    r = sum(t ** (2 * k) / (2 * k + 1) for k in range(1, 30))
    z = q * q
    assert np.max(np.abs(z * horner(c[1:8], z) - r)) <= 5.5e-18
    ln2 = LD("0.693147180559945309417232121458176568")
    assert abs(c[8] + c[9] + 2 * ln2) <= 2 ** -62
    assert all(float(LD(e) * c[8]) == LD(e) * c[8] for e in range(-24, 1))  # exact in FP64


def test_sine_and_cosine():
    """X = 2 pi 2^-24 x for |x| <= 2^21: sin X = X + X v s(v) with v = x^2 to
    2e-18, cos X = 1 + v c1 + v^2 c(v) to 2e-17 (as printed, to half a digit)."""
    c = constants("turn")
    sin, cos = c[:7], c[10:16]
    x = np.concatenate([np.linspace(LD(0), LD(2 ** 21), 200_001), LD(2) ** np.arange(0, 22)]).round()
    pi = LD("3.14159265358979323846264338327950288")
    X, v = x * (2 * pi / 2 ** 24), x * x
    series = sum(LD(-1) ** k * X ** (2 * k) / np.prod(np.arange(2, 2 * k + 2, dtype=LD)) for k in range(1, 14))
    assert np.max(np.abs(v * horner(sin, v) - series)) <= 2.5e-18  # sin X / X - 1
    assert abs(c[7] + c[8] - 2 * pi / 2 ** 24) <= 2.0 ** -84 and c[7] == c[9]
    series = sum(LD(-1) ** k * X ** (2 * k) / np.prod(np.arange(1, 2 * k + 1, dtype=LD)) for k in range(1, 14))
    assert c[16] == c[17]
    assert np.max(np.abs(v * c[16] + v * v * horner(cos, v) - series)) <= 2.5e-17
