"""The byte-digit arithmetic of the matrix-unit base conversion, in exact integers (no GPU).

A centred source word and a centred constant are written in signed bytes; the 32-bit products'
sums, the partial sums taken in 32 and 64 bits, and the two reductions must stay in range and give
sum_s y_s c_s mod q for the largest words and constants that eight sources can have.
"""
import math
import random

import pytest

BIAS = 0x8080808080808080
M64 = 1 << 64


def signed_bytes(y):
    """the kernel's form: (y + BIAS) xor BIAS as eight signed bytes"""
    w = ((y % M64) + BIAS) % M64 ^ BIAS
    d = [(w >> (8 * i)) & 255 for i in range(8)]
    return [v - 256 if v > 127 else v for v in d]


def centred(v, q):
    v %= q
    return v - q if v > (q - 1) // 2 else v


def column_sums(ys, cs, q):
    """a_e = sum over sources and bytes of byte e of the constant times the source's byte"""
    a = [0] * 8
    for y, c in zip(ys, cs):
        yd = signed_bytes(y)
        assert sum(d << (8 * i) for i, d in enumerate(yd)) == y
        for d in range(8):
            wd = signed_bytes(centred(c << (8 * d), q))
            for e in range(8):
                a[e] += yd[d] * wd[e]
    return a


def cases(q, seed):
    rng = random.Random(seed)
    top = (1 << 59) - 1
    edge = [top, -top, 0x7f7f7f7f7f7f7f, -0x8080808080808, 0, 1, -1]
    for _ in range(40):
        ns = rng.randint(1, 8)
        yield ([rng.choice(edge + [rng.randint(-top, top)]) for _ in range(ns)],
               [rng.choice([0, 1, q - 1, q // 2, q // 2 + 1, rng.randrange(q)]) for _ in range(ns)])
    yield [top] * 8, [q // 2] * 8
    yield [-top] * 8, [q // 2 + 1] * 8


@pytest.mark.parametrize("q", [(1 << 46) - 21, (1 << 45) - 55, (1 << 43) - 57, (1 << 43) + 29, (1 << 30) - 35, 786433])
def test_fp64_targets(q):
    for ys, cs in cases(q, q):
        a = column_sums(ys, cs, q)
        assert all(abs(v) <= 1 << 20 for v in a) and a[6] == a[7] == 0
        p = [a[0] + (a[1] << 8), a[2] + (a[3] << 8), a[4] + (a[5] << 8)]
        assert all(abs(v) < 1 << 31 for v in p)
        # the kernel's doubles: p2 2^32 and p0 + 2^16 p1 are exact, the quotient within one of the
        # rounded one, the remainder exact in one FMA
        qinv = 1.0 / q
        p2 = float(p[2]) * 4294967296.0
        c = round(p2 * qinv)
        r = p[2] * (1 << 32) - int(c) * q
        assert abs(r) <= q // 2 + 1 and float(r) == r
        lo = p[0] + (p[1] << 16)
        assert abs(lo) < 1 << 45 and abs(r + lo) < 1 << 53
        x = r + lo
        if q < 1 << 43:
            x -= round(float(x) * qinv) * q
        assert abs(x) < 4 * q
        assert (x - sum(y * c for y, c in zip(ys, cs))) % q == 0


@pytest.mark.parametrize("q", [(1 << 60) - 93, (1 << 46) + 15, (1 << 47) - 115, (1 << 59) + 131])
def test_integer_targets(q):
    w = (1 << 32) % q
    w_sh = (w << 64) // q
    off = -(1 << 77) % q
    if off < 1 << 45:
        off += q
    for ys, cs in cases(q, q):
        a = column_sums(ys, cs, q)
        assert all(abs(v) <= 1 << 20 for v in a)
        lo = a[0] + (a[1] << 8) + ((a[2] + (a[3] << 8)) << 16)
        hi = a[4] + (a[5] << 8) + ((a[6] + (a[7] << 8)) << 16)
        assert abs(lo) < 1 << 45 and abs(hi) < 1 << 45
        h = hi + (1 << 45)
        r = h * w - ((h * w_sh) >> 64) * q
        assert 0 <= r < 2 * q
        v = r + lo + off
        assert 0 <= v < 4 * q and v < M64
        assert (v - sum(y * c for y, c in zip(ys, cs))) % q == 0
    assert math.gcd(q, 2) == 1
