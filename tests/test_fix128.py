"""The device encoder's fixed-point transform is no further from the exact one than the 113-bit transform that it
stands in for: both run on the CPU, in the arithmetic of the kernels, against integers of 240 bits."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BITS = 240
ONE = 1 << BITS


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("fix128") / "fix128_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-o", exe, os.path.join(ROOT, "tests", "fix128_check.cpp")])
    return exe


def mul(a, b):
    return a * b + (ONE >> 1) >> BITS


def arctan_inverse(x):
    t, s, k = ONE * 1024 // x, 0, 0  # ten guard bits
    while t:
        s += (-t if k & 1 else t) // (2 * k + 1)
        t //= x * x
        k += 1
    return s


def cis(m):
    """(cos, sin)(pi k / m) for k < 2 m"""
    angle = (16 * arctan_inverse(5) - 4 * arctan_inverse(239)) // 1024 // m
    c, s, t, k = 0, 0, ONE, 0
    while t:
        if k & 1:
            s += -t if k & 2 else t
        else:
            c += -t if k & 2 else t
        k += 1
        t = mul(t, angle) // k
    out = [(ONE, 0)]
    for _ in range(2 * m - 1):
        a, b = out[-1]
        out.append((mul(a, c) - mul(b, s), mul(a, s) + mul(b, c)))
    return out


def exact(vals, log_n):
    """N / scale times the unrounded coefficients, times 2^240"""
    n = 1 << log_n
    table = cis(n)  # exp(i pi k / N)
    xr, xi = [0] * n, [0] * n
    power = 1
    for j in range(n // 2):
        num, den = float(vals[j % len(vals)]).as_integer_ratio()
        assert ONE % den == 0
        xr[(power - 1) // 2] = xr[(2 * n - power - 1) // 2] = num * (ONE // den)
        power = power * 5 % (2 * n)
    half, stride = n // 2, 1
    while half:
        for b in range(0, n, 2 * half):
            for j in range(b, b + half):
                ur, ui = xr[j] - xr[j + half], xi[j] - xi[j + half]
                xr[j] += xr[j + half]
                xi[j] += xi[j + half]
                c, s = table[2 * (j - b) * stride]
                xr[j + half], xi[j + half] = mul(ur, c) + mul(ui, s), mul(ui, c) - mul(ur, s)
        half, stride = half // 2, stride * 2
    at = [int(format(i, f"0{log_n}b")[::-1], 2) for i in range(n)]
    return [mul(xr[at[i]], table[i][0]) + mul(xi[at[i]], table[i][1]) for i in range(n)]


@pytest.mark.parametrize("log_n", [8, 10, 12, 13])
@pytest.mark.parametrize("spread", [0, 40])
def test_error_against_113_bits(driver, log_n, spread):
    rng = np.random.default_rng(log_n + spread)
    half = 1 << (log_n - 1)
    for count in (half, 16):
        vals = rng.uniform(-1, 1, count) * 2.0 ** -rng.integers(0, spread + 1, count)
        out = subprocess.run([driver, str(log_n)], input="\n".join(repr(float(v)) for v in vals), text=True,
                             capture_output=True, check=True, timeout=120).stdout.splitlines()
        shift, want = int(out[0]), exact(vals, log_n)
        fixed = float113 = 0
        for line, w in zip(out[1:], want):
            y, m, e = line.split()
            fixed = max(fixed, abs((int(y, 16) << (BITS - shift)) - w))
            m, e = int(m, 16), int(e) + BITS
            float113 = max(float113, abs((m << e if e >= 0 else m >> -e) - w))
        bits = [np.log2(x / max(map(abs, want))) for x in (fixed, float113)]
        print(f"[fix128] N=2^{log_n} {count} values over 2^-{spread}: worst error 2^{bits[0]:.1f} of the largest "
              f"coefficient, 113 bits 2^{bits[1]:.1f}")
        assert fixed <= float113
