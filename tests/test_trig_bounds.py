"""The trigonometric fast path's error (cr_f32_trig.h), replayed with every binary64
operation rounded to nearest and compared with the exact values (CPU): sine and cosine
within 2^-46 of their value, 2^-47.6 away from the zeros of both, and their quotient
within 2^-45.9, which the rounding test's 512 units in the last place cover."""
import os
import random
import re
import struct
from fractions import Fraction as Fr

import mpmath as mp
import pytest

from test_trig_reduction import HDR, ROOT, arr, f32, fma, hdr, reduce, rows  # noqa: F401


@pytest.fixture(scope="module")
def consts(hdr):  # noqa: F811
    body = re.search(r"SINCOS_T\[16\] = \{(.*?)\n\};", hdr, flags=re.S).group(1)
    t = [[float.fromhex(v.strip()) for v in r.split(",")] for r in re.findall(r"\{([^{}]*)\}", body)]
    return {"t": t, "s": [float(v) for v in arr(hdr, "SIN_F")], "c": [float(v) for v in arr(hdr, "COS_F")]}


def core(x, rows, K):  # noqa: F811
    """(sin x, cos x, j) as the kernel evaluates them, x > 0"""
    q, f = reduce(x, rows)
    f2 = f * f
    s, c = K["s"], K["c"]
    sr = f * fma(fma(fma(s[3], f2, s[2]), f2, s[1]), f2, s[0])
    cm1 = f2 * fma(fma(c[2], f2, c[1]), f2, c[0])
    row, odd = K["t"][q & 15], (q >> 4) & 1
    T1, T2 = (row[2], row[0]) if odd else (row[0], row[2])
    srq = -sr if odd else sr
    sn = T1 + fma(T1, cm1, T2 * srq)
    cs = T2 + fma(T2, cm1, -(T1 * srq))
    return (-sn if q & 32 else sn), (-cs if (q ^ (q << 1)) & 32 else cs), q & 15


def worst(points, rows, K):  # noqa: F811
    """log2 of the largest relative error of sine or cosine at j = 0, elsewhere, and of
    the tangent's exact quotient"""
    e = [mp.mpf(0)] * 3
    with mp.workprec(420):
        for x in points:
            s, c, j = core(x, rows, K)
            S, C = mp.sin(mp.mpf(x)), mp.cos(mp.mpf(x))
            d = max(abs(s / S - 1), abs(c / C - 1))
            k = 0 if j == 0 else 1
            e[k] = max(e[k], d)
            e[2] = max(e[2], abs(mp.mpf(s) / mp.mpf(c) * C / S - 1))
        return [float(mp.log(v, 2)) for v in e]


def test_errors_and_the_rounding_test(rows, consts):  # noqa: F811
    r = random.Random(5)
    points = [f32(r.randrange(0x39800000, 0x7f800000)) for _ in range(3000)]
    points += [f32(r.randrange(0x3f000000, 0x43000000)) for _ in range(3000)]
    # next to the zeros: the binary32 numbers around k pi/2
    with mp.workprec(200):
        for k in list(range(1, 400)) + [r.randrange(1, 1 << 22) for _ in range(600)]:
            b = float(mp.mpf(k) * mp.pi / 2)
            n = struct.unpack("<I", struct.pack("<f", b))[0]
            points += [f32(n - 1), f32(n), f32(n + 1)]
    near, far, tan = worst(points, rows, consts)
    assert near <= -46 and far <= -47.6, (near, far)
    # div_fast adds 2^-52
    total = 2.0 ** tan + 2.0 ** -52
    assert total <= 2.0 ** -45.9
    # relative 2^-45.9 is below 2^-45.9 2^53 units in the last place; the test is sound
    # below E + 1 of them
    text = open(os.path.join(ROOT, "paper_2605_15547_amd", "csrc", "cr_f32_trig.h")).read()
    E = int(re.search(r"TRIG_TEST_E = (\d+);", text).group(1))
    assert Fr(2) ** 53 * Fr(2.0 ** -45.9) < E + 1
