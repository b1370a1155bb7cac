"""The register column passes' lazy bounds, in exact integers (no GPU): the reduction that feeds them, as the
kernel takes it with the short quotient, and every stage of the forward and inverse schedules, whole columns
and columns spread over four or two lane groups, from the largest values that each stage can meet."""
import random

import pytest

from test_byte_conversion import cases, column_sums
from test_lean_butterfly import M, mul_lean, red16

QS = [(1 << 60) - 93, (1 << 46) + 15, (1 << 47) - 115, (1 << 59) + 131]


@pytest.mark.parametrize("q", QS)
def test_conversion_enters_below_6q(q):
    w = (1 << 32) % q
    off = -(1 << 77) % q
    off += q if off < 1 << 45 else 0
    for ys, cs in cases(q, q):
        a = column_sums(ys, cs, q)
        lo = a[0] + (a[1] << 8) + ((a[2] + (a[3] << 8)) << 16)
        hi = a[4] + (a[5] << 8) + ((a[6] + (a[7] << 8)) << 16)
        assert 0 <= lo + off < 2 * q and 0 <= hi + (1 << 45)
        v = mul_lean(lo + off, hi + (1 << 45), w, (w << 64) // q, q)
        assert v < 6 * q and (v - sum(y * c for y, c in zip(ys, cs))) % q == 0


class Words:
    """values and the bounds that the kernels' comments give for them, in units of q; every sum fits 64 bits"""

    def __init__(self, q, seed):
        self.q, self.rng = q, random.Random(seed)

    def below(self, units):
        return self.rng.choice([0, units * self.q - 1, units * self.q - 1 - self.rng.randrange(self.q)])

    def check(self, v, units):
        assert units <= 16 and 0 <= v < units * self.q <= M + 1, (v / self.q, units)
        return v, units

    def product(self, u, a, units):
        w = self.rng.choice([0, 1, self.q - 1, self.rng.randrange(self.q)])
        assert 0 <= a <= M
        return self.check(mul_lean(u, a, w, (w << 64) // self.q, self.q), units)

    def reduced(self, v, units):
        self.check(v, units)
        return red16(v, self.q), 2


@pytest.mark.parametrize("q", QS)
@pytest.mark.parametrize("l1", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("split", [1, 2, 4])
def test_forward_schedule(q, l1, split):
    for seed in range(8):
        t, n = Words(q, seed), 1 << l1
        x = [(t.below(6), 6) for _ in range(n)]
        bound = 6
        for st in range(l1):
            d = n >> (st + 1)
            red = bound + 4 > 16
            if d >= split:
                bound = (2 if red else bound) + 4
            for i in range(1 << st):
                for j in range(2 * i * d, 2 * i * d + d):
                    if d < split:  # both lanes run a product, the lower one by one
                        a, b = t.product(0, x[j][0], 4)[0], t.product(0, x[j + d][0], 4)[0]
                        x[j], x[j + d] = t.check(a + b, 8), t.check(a + 4 * q - b, 8)
                        continue
                    u, ub = t.reduced(*x[j]) if red else x[j]
                    s = t.product(u, x[j + d][0], ub + 4)
                    x[j], x[j + d] = s, t.check(2 * u + 4 * q - s[0], ub + 4)
                    assert s[1] <= bound
        assert all(v < 16 * q for v, _ in x)


@pytest.mark.parametrize("q", QS)
@pytest.mark.parametrize("l1", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("split", [1, 2, 4])
def test_inverse_schedule(q, l1, split):
    for seed in range(8):
        t, n = Words(q, seed), 1 << l1
        x = [(t.below(4), 4) for _ in range(n)]
        for st in range(l1 - 1, -1, -1):
            d = n >> (st + 1)
            for i in range(1 << st):
                for j in range(2 * i * d, 2 * i * d + d):
                    (u, ub), (v, vb) = x[j], x[j + d]
                    if split > 1:
                        assert ub <= 4 and vb <= 4
                        if d < split:
                            x[j], x[j + d] = t.product(0, u + v, 4), t.product(0, u + 4 * q - v, 4)
                        else:
                            s = u + v
                            x[j], x[j + d] = t.check(s - 4 * q if s >= 4 * q else s, 4), t.product(0, u - v + 4 * q, 4)
                        continue
                    if ub == 16:
                        u, v, ub, vb = t.reduced(u, 16)[0], t.reduced(v, 16)[0], 4, 4
                    assert ub == vb
                    x[j] = t.check(u + v, 2 * ub)
                    x[j + d] = t.product(0, u + ub * q - v, 4)
        assert all(v < 16 * q for v, _ in x)
