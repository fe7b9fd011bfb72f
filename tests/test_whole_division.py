"""The samplers divide by whole numbers with one product and one residual
correction.  Its claim, that the result is the correctly rounded quotient for
any reciprocal within a few ulp, checked in exact arithmetic (float() of a
Fraction rounds correctly, so a fused multiply-add is the float of the exact
value)."""
import math
from fractions import Fraction as F

import numpy as np


def fma(a, b, c):
    return float(F(a) * F(b) + F(c))


def quotient(a, x, y):
    q = a * y
    return fma(fma(-x, q, a), y, q)


def test_correctly_rounded_for_any_near_reciprocal():
    rng = np.random.default_rng(1)
    for i in range(20000):
        x = float(rng.integers(1, 65) if i % 2 else rng.integers(1, 2**31 - 1))
        a = math.ldexp(1.0 + rng.random(), int(rng.integers(-300, 300)))
        if i % 3 == 0:  # quotients next to the midpoint of two doubles
            mid = F(math.ldexp(1.0 + rng.random(), 0)) + F(1, 2**53)
            a = float(mid * F(x))
        y = 1.0 / x
        for _ in range(int(rng.integers(0, 4))):
            y = math.nextafter(y, math.inf if i % 5 else 0.0) if hasattr(math, "nextafter") else float(
                np.nextafter(y, np.inf if i % 5 else 0.0))
        assert quotient(a, x, y) == a / x, (a, x, y)
