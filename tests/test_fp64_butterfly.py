"""The FP64 modular product of the transforms' butterflies, emulated with exact integers (no GPU):
hi = fl(a w), lo the exact rest, c = rint(fl(hi fl(1/q))), result hi - c q + lo.  It is a w mod q exactly, and below
0.95 q in magnitude up to the largest operand a forward transform reaches (19.3 q after 15 stages from
4 q, each adding less than 0.95 q), so the bound is its own proof for every stage."""
import random

import pytest


def mulmod(a, w, q):
    hi = float(a * w)  # Python rounds the exact product once, as v_mul_f64 does
    lo = a * w - int(hi)
    assert float(lo) == lo  # what the FMA returns exactly
    c = round(hi * (1.0 / q))  # half to even, as v_rndne_f64
    r = int(hi) - c * q
    assert float(r) == r  # the FMA's remainder needs no rounding
    assert float(r + lo) == r + lo
    return r + lo


@pytest.mark.parametrize("q", [(1 << 46) - 21, (1 << 46) - 2 ** 17 + 1, (1 << 45) - 55, (1 << 44) + 7, (1 << 40) - 87, 786433])
def test_product_is_exact_and_bounded(q):
    rng = random.Random(q)
    top = int(19.3 * q)
    for i in range(20000):
        a = rng.choice([top, -top, top - rng.randrange(q), rng.randrange(-top, top + 1)])
        w = rng.choice([q - 1, q // 2, 1, rng.randrange(1, q)])
        r = mulmod(a, w, q)
        assert (r - a * w) % q == 0
        assert abs(r) < 0.95 * q
    # operands whose quotient is next to a half: the rounded quotient may fall either way
    for i in range(2000):
        w = rng.randrange(q // 2, q)
        k = rng.randrange(19 * w // q + 1)
        a = ((2 * k + 1) * q // 2 + rng.randrange(-3, 4)) // w
        if abs(a) <= top:
            assert abs(mulmod(a, w, q)) < 0.95 * q
