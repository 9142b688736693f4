"""The fp32 GeLU's fitted constants, read from the kernel source: each fit against the function it stands for, and the
kernel's formula, evaluated in fp32, against the plain form 0.5 (1 + erf(z / sqrt 2)) with a correctly rounded erf."""
import math
import os
import re

import numpy as np
import pytest
from scipy.special import erf, erfc, erfcx

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2109_10465_amd", "csrc", "expert_gemm.hip")
f = np.float32


def constants():
    text = open(SRC).read()
    out = {}
    for name in ("CENTRE", "MILLS_NUM", "MILLS_DEN"):
        body, = re.findall(r"constexpr float %s\[\d\] = \{([^}]*)\}" % name, text)
        out[name] = [f(v.strip().rstrip("f")) for v in body.split(",")]
    for name in ("LH", "PHI0", "PHI0_LN2"):
        v, = re.findall(r"\b%s = (-?[0-9.e+-]+)f" % name, text)
        out[name] = f(v)
    return out


K = constants()
EDGE = 1.0625


def poly64(c, x):
    return sum(float(v) * x ** i for i, v in enumerate(c))


def test_fits():
    z = np.linspace(1e-6, EDGE, 200001)
    # within a tenth of the rounding of 1/2 (6e-8 / 2)
    assert np.abs(z * poly64(K["CENTRE"], z * z) - 0.5 * erf(z / math.sqrt(2.0))).max() <= 3e-9
    t = np.linspace(EDGE, 13.5, 200001)
    mills = math.sqrt(math.pi / 2.0) * erfcx(t / math.sqrt(2.0))
    # the fit's 2.6e-8 and the roundings of the coefficients above and below, 2^-24 each at most
    assert np.abs(poly64(K["MILLS_NUM"], t) / poly64(K["MILLS_DEN"], t) / mills - 1.0).max() <= 2.6e-8 + 2 * 2.0 ** -24
    assert K["LH"] == f(-math.log2(math.e) / 2.0)
    assert K["PHI0"] == f(1.0 / math.sqrt(2.0 * math.pi)) and K["PHI0_LN2"] == f(math.log(2.0) / math.sqrt(2.0 * math.pi))


def fma(a, b, c):
    return f(np.asarray(a, np.longdouble) * np.asarray(b, np.longdouble) + np.asarray(c, np.longdouble))


def horner(c, x):
    p = np.full_like(x, c[-1])
    for v in c[-2::-1]:
        p = fma(p, x, v)
    return p


def kernel_form(z):
    t = np.minimum(np.abs(z), f(16))
    s = f(t * t)
    e = f(s * K["LH"])
    rest = fma(s, K["LH"], -e)
    pdf = f(f(np.exp2(e.astype(np.float64))) * fma(rest, K["PHI0_LN2"], K["PHI0"]))
    q = f(f(horner(K["MILLS_NUM"], t) * pdf) * f(1.0 / horner(K["MILLS_DEN"], t).astype(np.float64)))
    cdf = np.where(t < f(EDGE), fma(z, horner(K["CENTRE"], s), f(0.5)), np.where(z >= 0, f(f(1) - q), q))
    return f(z * cdf), fma(z, pdf, cdf)


def plain_form(z):
    cdf = f(f(0.5) * f(f(1) + f(erf(f(z * f(math.sqrt(0.5))).astype(np.float64)))))
    pdf = f(np.exp(f(f(f(-0.5) * z) * z).astype(np.float64)))
    return f(z * cdf), f(cdf + f(f(z * K["PHI0"]) * pdf))


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("lo,hi", [(0, 0.5), (0.5, 1), (1, 1.5), (1.5, 2), (2, 3), (3, 5), (5, 8)])
def test_error_is_no_larger_than_that_of_erf_and_exp(lo, hi, sign):
    z = f(sign * np.random.default_rng(1).uniform(lo, hi, 200000))
    z64 = z.astype(np.float64)
    cdf = 0.5 * erfc(-z64 / math.sqrt(2.0))
    exact = z64 * cdf, cdf + z64 * np.exp(-0.5 * z64 * z64) / math.sqrt(2.0 * math.pi)
    for new, old, want in zip(kernel_form(z), plain_form(z), exact):
        en, eo = new - want, old - want
        # 1 % for the sample; the largest single error of either is one rounding event of many
        assert np.sqrt((en ** 2).mean()) <= 1.01 * np.sqrt((eo ** 2).mean())
        assert np.abs(en).max() <= 1.25 * np.abs(eo).max()
