"""The trigonometric fast path's reduction (cr_f32_trig.h, trig_fast_core) replayed
in exact rational arithmetic with every binary64 operation rounded to nearest (CPU),
with the constants read back from the generated header."""
import os
import random
import re
import struct
from fractions import Fraction

import mpmath as mp
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HDR = os.path.join(ROOT, "paper_2605_15547_amd", "csrc", "cr_consts.h")
MAGIC = 1.5 * 2.0 ** 52


@pytest.fixture(scope="module")
def hdr():
    with open(HDR) as f:
        return f.read()


@pytest.fixture(scope="module")
def rows(hdr):
    m = re.search(r"TRIG_RED\[16\] = \{(.*?)\n\};", hdr, flags=re.S)
    out = [[float.fromhex(v.strip()) for v in r.split(",")] for r in re.findall(r"\{([^{}]*)\}", m.group(1))]
    assert len(out) == 16
    return out


def arr(txt, name):
    m = re.search(r"\b%s\[\d+\] = \{([^}]*)\}" % re.escape(name), txt)
    return [float.fromhex(v.strip()) for v in m.group(1).split(",")]


def frac(x):
    """an mpf as an exact fraction"""
    s, man, e, _ = mp.mpf(x)._mpf_
    return Fraction(-man if s else man) * Fraction(2) ** e


with mp.workprec(700):
    N_PER_X = frac(32 / mp.pi)  # 32/pi to 700 bits


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))  # Fraction -> float rounds to nearest even


def reduce(x, rows):
    """(k mod 64, f) as the kernel computes them"""
    bits = struct.unpack("<I", struct.pack("<f", x))[0]
    w = rows[max(bits >> 26, 16) - 16]
    p2 = x * w[1]
    assert Fraction(p2) == Fraction(x) * Fraction(w[1])
    t = fma(x, w[0], p2) + MAGIC
    kd = t - MAGIC
    d = fma(x, w[0], -kd)
    assert Fraction(d) == Fraction(x) * Fraction(w[0]) - Fraction(kd)  # exact
    f = fma(x, w[2], d + p2)
    return struct.unpack("<Q", struct.pack("<d", t))[0] & 63, f


def f32(bits):
    return struct.unpack("<f", struct.pack("<I", bits))[0]


def check(x, rows):
    q, f = reduce(x, rows)
    n = Fraction(x) * N_PER_X
    d = (n - q) / 64  # f is N - k, k = q mod 64
    want = (d - round(d)) * 64
    assert abs(f) <= 0.5 + 2.0 ** -17
    # the truth is known to 2^-560 here
    assert abs(Fraction(f) - want) <= Fraction(2) ** -52 * abs(want) + Fraction(2) ** -74, (x.hex(), q, f)


def test_reduction_of_random_arguments(rows):
    r = random.Random(1)
    for _ in range(20000):
        check(f32(r.randrange(0x39800000, 0x7f800000)), rows)


def test_reduction_at_row_edges(rows):
    r = random.Random(2)
    for e in range(115, 255):
        for m in [0, 1, 0x7fffff, 0x7ffffe] + [r.randrange(1 << 23) for _ in range(20)]:
            check(f32((e << 23) | m), rows)


def nearest(E):
    """A lower bound of |M 2^E 32/pi - k| / 16 over 0 < M < 2^24, k a multiple of 16
    (the distance of x 2/pi to the integers), by the continued fraction of 2^E 2/pi: no
    M below a denominator comes closer than the convergent before it."""
    with mp.workprec(700):
        a = frac(mp.mpf(2) ** E * 2 / mp.pi) % 1
    best, h0, h1, y = Fraction(1), (1, 0), (0, 1), a
    while True:  # convergents p/q of a
        c = y.numerator // y.denominator
        h0, h1 = (c * h0[0] + h1[0], c * h0[1] + h1[1]), h0
        q = h0[1]
        if q >= 1 << 24:
            return best
        if q:
            best = min(best, abs(q * a - h0[0]))
        y = y - c
        if y == 0:
            return best
        y = 1 / y


def test_no_argument_comes_closer_than_2_to_minus_30_to_a_zero(rows):
    """Arguments of at least 2^-12 (smaller ones are special cases): |x - k pi/2| >=
    2^-30 for k != 0, so sin r and cos r of the j = 0 rows are normal numbers known to
    the relative bound of the rounding test.  (k = 0 is x itself.)"""
    worst = min(nearest(E) for E in range(-23, 105))
    assert worst * Fraction(11, 7) > Fraction(1, 1 << 30), float(worst)


def test_polynomials_in_f(hdr):
    """SIN_F and COS_F are SIN_S2 and COS_C2 scaled to f = r 32/pi, each coefficient to
    half an ulp, and the bounds of the latter hold for the reduction's whole range."""
    from paper_2605_15547_amd.gen import bounds as B
    s, c = arr(hdr, "SIN_F"), arr(hdr, "COS_F")
    with mp.workprec(300):
        p = mp.pi / 32
        want_s = [p] + [mp.mpf(v) * p ** (2 * k + 3) for k, v in enumerate(arr(hdr, "SIN_S2"))]
        want_c = [mp.mpf(v) * p ** (2 * k + 2) for k, v in enumerate(arr(hdr, "COS_C2"))]
        for got, want in ((s, want_s), (c, want_c)):
            assert len(got) == len(want)
            for g, w in zip(got, want):
                assert abs(mp.mpf(g) - w) <= abs(w) * mp.mpf(2) ** -53
    rho = mp.pi / 64 * (1 + mp.mpf(2) ** -16)
    assert B.log2b(B.sup_bound(B.sin_minus_r([mp.mpf(v) for v in arr(hdr, "SIN_S2")], rho))) <= -64
    assert B.log2b(B.sup_bound(B.cos_minus_1([mp.mpf(v) for v in arr(hdr, "COS_C2")], rho))) <= -56
