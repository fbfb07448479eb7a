"""The binary64 log main path (cr_f64.h, log64_fast) with the constants of the generated
header: table identities, the polynomial's proven bound, and the evaluation replayed with
every binary64 operation rounded to nearest against the exact logarithm (CPU)."""
import math
import os
import random
import re
from fractions import Fraction as Fr

import mpmath as mp
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HDR = os.path.join(ROOT, "paper_2605_15547_amd", "csrc", "cr_consts.h")

from paper_2605_15547_amd.gen import bounds as B  # noqa: E402


@pytest.fixture(scope="module")
def K():
    txt = open(HDR).read()

    def rows(name):
        m = re.search(r"%s\[16\] = \{(.*?)\n\};" % name, txt, flags=re.S)
        return [[float.fromhex(v.strip()) for v in r.split(",")] for r in re.findall(r"\{([^{}]*)\}", m.group(1))]

    def const(name):
        return float.fromhex(re.search(r"#define %s \(([^)]*)\)" % name, txt).group(1))
    S = re.search(r"LOG64_S3\[\d+\] = \{([^}]*)\}", txt).group(1)
    return {"r1": rows("LOG64_R1"), "r2": rows("LOG64_R2"), "hi": const("LOG64_LN2_HI"),
            "lo": const("LOG64_LN2_LO"), "S": [float.fromhex(v.strip()) for v in S.split(",")]}


def fma(a, b, c):
    return float(Fr(a) * Fr(b) + Fr(c))


def setup(x):
    f, e = math.frexp(x)  # [1/2, 1)
    m, e = 2 * f, e - 1
    j = int((m - 1) * 16)
    return (m / 2, e + 1, j) if j >= 8 else (m, e, j)


def replay(x, K):
    """(y as a fraction, tail, Ah)"""
    m, e, j = setup(x)
    A = K["r1"][j]
    k = int(fma(m * A[0], 128.0, 1.5 * 2.0 ** 52) - 1.5 * 2.0 ** 52)
    assert 124 <= k <= 136
    Bk = K["r2"][k % 16]
    C = A[0] * Bk[0]
    assert Fr(C) == Fr(A[0]) * Fr(Bk[0])
    ph = m * C
    pl = fma(m, C, -ph)
    t = (ph - 1.0) + pl
    tl = pl - (t - (ph - 1.0))
    assert Fr(t) + Fr(tl) == Fr(m) * Fr(C) - 1  # exact
    qh = t * (-0.5 * t)
    ql = fma(-t, tl, fma(t, -0.5 * t, -qh))
    s = K["S"][-1]
    for c in K["S"][-2::-1]:
        s = fma(s, t, c)
    tail = (qh * t) * s
    lh = t + qh
    ll = qh - (lh - t)
    Ah = fma(e, K["hi"], A[1] + Bk[1])
    assert Fr(Ah) == e * Fr(K["hi"]) + Fr(A[1]) + Fr(Bk[1])  # exact
    Al = fma(e, K["lo"], A[2] + Bk[2])
    yh = Ah + lh
    bb = yh - Ah
    yl = (Ah - (yh - bb)) + (lh - bb)
    lo = yl + ((ll + (tl + (ql + tail))) + Al)
    return Fr(yh) + Fr(lo), tail, yh, t


def check(x, K):
    y, tail, yh, t = replay(x, K)
    assert abs(t) < 2.0 ** -7.9
    with mp.workprec(260):
        exact = mp.log(mp.mpf(x))
        err = abs(mp.mpf(y.numerator) / mp.mpf(y.denominator) - exact)
        assert err <= abs(mp.mpf(tail)) * mp.mpf(2) ** -49 + abs(mp.mpf(yh)) * mp.mpf(2) ** -78, x.hex()
        return float(err / (abs(mp.mpf(tail)) * mp.mpf(2) ** -49 + abs(mp.mpf(yh)) * mp.mpf(2) ** -78))


def test_tables(K):
    with mp.workprec(400):
        for rows in (K["r1"], [r for i, r in enumerate(K["r2"]) if i <= 8 or i >= 12]):
            for c, h, l, _ in rows:
                assert (h * 2.0 ** 42).is_integer()
                assert abs(mp.mpf(h) + mp.mpf(l) + mp.log(mp.mpf(c))) <= mp.mpf(2) ** -96
        assert (K["hi"] * 2.0 ** 42).is_integer()
        assert abs(mp.mpf(K["hi"]) + mp.mpf(K["lo"]) - mp.log(2)) <= mp.mpf(2) ** -96
    assert K["r2"][0][:3] == [1.0, 0.0, 0.0] and K["r1"][0][:3] == [1.0, 0.0, 0.0]


def test_polynomial(K):
    lim = mp.mpf("0.00404")
    assert B.log2b(B.sup_bound(B.log64_cubic([mp.mpf(v) for v in K["S"]], -lim, lim))) <= -54.4


def test_replay_over_the_range(K):
    r = random.Random(3)
    worst = 0.0
    for _ in range(4000):
        worst = max(worst, check(math.ldexp(1 + r.random(), r.randrange(-1022, 1024)), K))
    for _ in range(4000):
        worst = max(worst, check(r.uniform(0.74, 1.52), K))
    assert worst < 1.0


def test_replay_near_one_and_at_the_rows_edges(K):
    r = random.Random(4)
    for _ in range(3000):
        check(1.0 + r.choice((-1, 1)) * 2.0 ** -r.uniform(8, 52), K)
    for j in range(16):
        for k in range(124, 137):
            m = (k + 0.5) / 128 / K["r1"][j][0]
            for d in (-2, -1, 0, 1, 2):
                x = m + d * 2.0 ** -52
                if setup(x)[2] == j and 0.75 <= x < 1.5:
                    check(x, K)
