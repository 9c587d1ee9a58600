"""The sum of up to eight products modulo a prime below 2^50 that the inner product of the key switch reduces once: its steps in
correctly rounded arithmetic, at the ends of their range."""
from fractions import Fraction
from itertools import product

import pytest

START = 3.0 * 2.0 ** 101


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def reduced(p, pairs, c0):
    pinv = 1.0 / p
    h, l = START, 0.0
    for x, k in pairs:
        n = fma(x, k, h)
        assert 2.0 ** 102 <= n < 2.0 ** 103
        left = fma(x, k, h - n)
        assert Fraction(left) == Fraction(x) * Fraction(k) + Fraction(h) - Fraction(n)  # nothing is lost
        l, h = l + left, n
    l += c0
    t = h - START
    r = fma(-float(round(Fraction(t * pinv))), p, t)
    assert abs(r) <= p * 1.01 + 2.0 ** 50 and abs(l) + abs(r) < 2.0 ** 53
    v = r + l
    return fma(-float(round(Fraction(v * pinv))), p, v)


@pytest.mark.parametrize("p", [(1 << 50) - 27, (1 << 49) + 1, (1 << 45) - 55, (1 << 36) - 5, (1 << 20) + 7])
@pytest.mark.parametrize("n", [1, 4, 8])
def test_sum_at_the_ends_of_its_range(p, n):
    e = float(p // 2)
    for sx, sk, odd, c in product((1, -1), (1, -1), (0, 1, 12345), (e, -e, 0.0)):
        pairs = [(sx * (e - odd), sk * (e - 2 * odd * (i % 2))) for i in range(n)]
        got = reduced(float(p), pairs, c)
        assert abs(got) <= p and (int(got) - sum(int(x) * int(k) for x, k in pairs) - int(c)) % p == 0
