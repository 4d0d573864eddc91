"""Host check of the push's cell quotient: two corrections by a correctly
rounded reciprocal give the rounded quotient, as the division does."""
from fractions import Fraction

import numpy as np


def _fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))  # one rounding


def _quotient(a, b):
    y = 1.0 / b
    q = a * y
    q = _fma(_fma(-q, b, a), y, q)
    return _fma(_fma(-q, b, a), y, q)


def test_quotient_is_the_rounded_one():
    rng = np.random.default_rng(5)
    b = np.concatenate([rng.uniform(1e-7, 1e-2, 2000), np.nextafter(2.0 ** -rng.integers(5, 20, 500), 1.0)])
    g = np.concatenate([rng.uniform(0, 1 << 20, 1500), rng.integers(0, 4096, 1000).astype(float)])
    a = g * b
    for d in (-2, -1, 0, 1, 2):  # next to whole quotients, where the cell changes
        x = a.copy()
        for _ in range(abs(d)):
            x = np.nextafter(x, np.inf if d > 0 else -np.inf)
        for ai, bi in zip(x.tolist(), b.tolist()):
            assert _quotient(ai, bi) == ai / bi, (ai, bi)
