"""GELU of the encoder on the host: the digits in the source against 64 bits, and the kernel's fp32 steps against those of the plain form."""
import math
import os
import re

import numpy as np

F = np.float32
SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2101_06983_amd", "csrc", "mlp.hip")
erf = np.vectorize(math.erf)
erfc = np.vectorize(math.erfc)


def digits(name):
    text = open(SRC).read()
    one = re.search(r"\b%s = ([-0-9.e]+)f" % name, text)
    many = re.search(r"\b%s\[\d+\] = \{([^}]*)\}" % name, text)
    return float(F(one.group(1))) if one else [float(F(x.strip().rstrip("f"))) for x in many.group(1).split(",")]


EDGE, SCALE, NEAR, FAR = digits("kPhiEdge"), digits("kPhiScale"), digits("kPhiNear"), digits("kPhiFar")


def fma(a, b, c):
    return (np.asarray(a, np.float64) * np.asarray(b, np.float64) + np.asarray(c, np.float64)).astype(F)


def mul(a, b):
    return np.asarray(a, F) * np.asarray(b, F)


def off(x, rng):   # a hardware result is up to half an ulp further off than the rounded one
    return (x * (1.0 + 2.0 ** -24 * rng.uniform(-1, 1, x.shape))).astype(F)


def kernel(h, rng):
    y, u = mul(h, h), np.abs(h)
    e = off(np.exp2(mul(y, F(-0.72134752)).astype(np.float64)).astype(F), rng)
    t = off((1.0 / fma(F(SCALE), u, F(1)).astype(np.float64)).astype(F), rng)
    p, q = np.full_like(h, F(NEAR[-1])), np.full_like(h, F(FAR[-1]))
    for c in NEAR[-2::-1]:
        p = fma(p, y, F(c))
    for c in FAR[-2::-1]:
        q = fma(q, t, F(c))
    tail = mul(mul(q, t), e)
    phi = np.where(u < F(EDGE), fma(h, p, F(0.5)), np.where(h >= 0, F(1) - tail, tail))
    return mul(h, phi), fma(mul(h, F(0.3989422804014327)), e, phi)


def plain(h, rng):   # h (1 + erf(h / sqrt 2)) / 2 and its derivative
    one = F(1) + off(erf(mul(h, F(math.sqrt(0.5))).astype(np.float64)).astype(F), rng)
    e = off(np.exp(mul(mul(F(-0.5), h), h).astype(np.float64)).astype(F), rng)
    return mul(mul(F(0.5), h), one), fma(mul(h, F(0.3989422804014327)), e, mul(F(0.5), one))


def exact(h):
    h = h.astype(np.float64)
    phi = 0.5 * erfc(-h / math.sqrt(2.0))
    return h * phi, phi + h * np.exp(-0.5 * h * h) / math.sqrt(2.0 * math.pi)


def test_the_fits_hold_what_the_source_says():
    u = np.linspace(0.0, EDGE, 20001)
    assert np.abs(0.5 + u * np.polyval(NEAR[::-1], u * u) - 0.5 * erfc(-u / math.sqrt(2.0))).max() < 3.6e-9
    u = np.linspace(EDGE, 14.0, 40001)
    t = 1.0 / (1.0 + SCALE * u)
    assert np.abs(np.exp(-0.5 * u * u) * t * np.polyval(FAR[::-1], t) / (0.5 * erfc(u / math.sqrt(2.0))) - 1.0).max() < 1.1e-7


def test_no_less_precise_than_the_plain_form():
    rng = np.random.default_rng(1)
    for s in (0.02, 0.1, 0.3, 0.6, 1.0, 2.0, 4.0):
        h = (rng.standard_normal(100000) * s).astype(F)
        for name, got, ref, want in zip(("gelu", "derivative"), kernel(h, rng), plain(h, rng), exact(h)):
            mine, theirs = (float(np.sqrt(((x - want) ** 2).mean())) for x in (got, ref))
            assert mine <= 1.02 * theirs, (s, name, mine, theirs)   # (2 %: the draw of the hardware's last bits)


def test_negative_arguments_keep_their_digits():
    rng = np.random.default_rng(2)
    for lo, hi, bound in ((-4.0, -0.01, 1.2e-6), (-8.0, -4.0, 3.5e-6), (-13.0, -8.0, 9e-6)):
        h = np.linspace(lo, hi, 50001).astype(F)
        assert np.abs(kernel(h, rng)[0] / exact(h)[0] - 1.0).max() < bound
