"""The integer butterflies' lazy bounds, in exact integers: the product with a short quotient and the
reduction below 16 q, at random and extreme operands, for primes of every width the ring takes."""
import random

import pytest

M = (1 << 64) - 1


def mul_lean(u, a, w, ws, q):
    h = (a >> 32) * (ws >> 32) + ((a >> 32) * (ws & 0xffffffff) >> 32) + ((a & 0xffffffff) * (ws >> 32) >> 32)
    return (u + a * w - h * q) & M


def red16(x, q):
    sh = max(q.bit_length() - 28, 0)
    c = (M // q) >> (32 - sh)
    assert c < 1 << 32 and x >> sh < 1 << 32
    return (x - ((x >> sh) * c >> 32) * q) & M


@pytest.mark.parametrize("bits", [20, 27, 28, 29, 33, 46, 47, 53, 59, 60])
def test_bounds(bits):
    rng = random.Random(bits)
    for q in {(1 << bits) - 1 - 2 * rng.randrange(1 << (bits - 6)) for _ in range(20)} | {(1 << (bits - 1)) + 1, (1 << bits) - 1}:
        top = min(16 * q, 1 << 64)
        for x in [0, 1, q - 1, q, 3 * q, 4 * q - 1, 8 * q, top - 1] + [rng.randrange(top) for _ in range(50)]:
            r = red16(x, q)
            assert r < 3 * q and r % q == x % q
        for w in [0, 1, q - 1, q // 2] + [rng.randrange(q) for _ in range(10)]:
            ws = (w << 64) // q
            for a in [0, q - 1, M, top - 1, (1 << 32) - 1, M ^ 0xffffffff] + [rng.randrange(1 << 64) for _ in range(20)]:
                v = mul_lean(0, a, w, ws, q)
                assert v < 4 * q and v % q == a * w % q
                # radix-8 growth: three stages from a reduced element stay below 16 q
                u = 11 * q - 1
                assert u + v < 16 * q <= 1 << 64 and u + 4 * q - v >= 0
