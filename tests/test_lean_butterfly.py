"""The integer butterflies' lazy bounds, in exact integers: the product with a short quotient and the
reduction below 16 q, at random and extreme operands, for primes of every width the ring takes."""
import random

import pytest

M = (1 << 64) - 1


def mul_lean(u, a, w, ws, q):
    h = (a >> 32) * (ws >> 32) + ((a >> 32) * (ws & 0xffffffff) >> 32) + ((a & 0xffffffff) * (ws >> 32) >> 32)
    return (u + a * w - h * q) & M


def red16(x, q):
    sh = q.bit_length() - 16
    c = (1 << (q.bit_length() + 16)) // q
    assert c < 1 << 32 and x >> sh < 1 << 20
    return (x - ((x >> sh) * c >> 32) * q) & M


LOW = (1 << 30) - 1


def redc60(c0, c1, c2, products, q):
    """column sums as 64-bit words: every step must fit them"""
    n = -pow(q, -1, 1 << 30) & LOW
    if products > 7:
        c2, c1 = c2 + (c1 >> 30), c1 & LOW
    m0 = c0 * n & LOW
    c0 += m0 * (q & LOW)
    c1 += m0 * (q >> 30) + (c0 >> 30)
    assert c0 <= M and c1 <= M and c0 & LOW == 0
    m1 = c1 * n & LOW
    c1 += m1 * (q & LOW)
    c2 += m1 * (q >> 30)
    assert c1 <= M and c1 & LOW == 0 and c2 + (c1 >> 30) <= M
    return c2 + (c1 >> 30)


@pytest.mark.parametrize("products", range(1, 9))
@pytest.mark.parametrize("bits", [20, 31, 45, 59, 60])
def test_two_digit_reduction(bits, products):
    rng = random.Random(100 * bits + products)
    for q in {(1 << bits) - 1 - 2 * rng.randrange(1 << (bits - 6)) for _ in range(20)} | {(1 << (bits - 1)) + 1, (1 << bits) - 1}:
        for k in range(30):
            xs, ys = ([q - 1] * products if k == 0 else [rng.randrange(q) for _ in range(products)] for _ in range(2))
            c0 = sum((x & LOW) * (y & LOW) for x, y in zip(xs, ys))
            c1 = sum((x & LOW) * (y >> 30) + (x >> 30) * (y & LOW) for x, y in zip(xs, ys))
            c2 = sum((x >> 30) * (y >> 30) for x, y in zip(xs, ys))
            assert max(c0, c1, c2) <= M
            r = redc60(c0, c1, c2, products, q)
            assert r < (products + 1) * q and (r << 60) % q == sum(x * y for x, y in zip(xs, ys)) % q


@pytest.mark.parametrize("bits", [20, 27, 28, 29, 33, 46, 47, 53, 59, 60])
def test_bounds(bits):
    rng = random.Random(bits)
    for q in {(1 << bits) - 1 - 2 * rng.randrange(1 << (bits - 6)) for _ in range(20)} | {(1 << (bits - 1)) + 1, (1 << bits) - 1}:
        top = min(16 * q, 1 << 64)
        for x in [0, 1, q - 1, q, 3 * q, 4 * q - 1, 8 * q, top - 1] + [rng.randrange(top) for _ in range(50)]:
            r = red16(x, q)
            assert r < q + q // 1024 + 1 and r % q == x % q
        for w in [0, 1, q - 1, q // 2] + [rng.randrange(q) for _ in range(10)]:
            ws = (w << 64) // q
            for a in [0, q - 1, M, top - 1, (1 << 32) - 1, M ^ 0xffffffff] + [rng.randrange(1 << 64) for _ in range(20)]:
                v = mul_lean(0, a, w, ws, q)
                assert v < 4 * q and v % q == a * w % q
                # radix-8 growth: three stages from a reduced element stay below 16 q
                u = 11 * q - 1
                assert u + v < 16 * q <= 1 << 64 and u + 4 * q - v >= 0
