"""Ranges of the forward transform's values, of which only those that the first stage of a step adds to are reduced between steps
(fold_first).  Limits: 2^53 for doubles, 7.5 2^60 for the signed integers of primes just below 2^60."""
from fractions import Fraction as F

import pytest


def steps(start, fold_start, product, folded, stages):
    """Largest value after each step of `stages[i]` stages; a step after the first, or any if fold_start, begins with the fold."""
    b, ends = start, []
    for i, n in enumerate(stages):
        x, y = (folded, b) if i or fold_start else (b, b)
        for _ in range(n):
            x = y = x + product(y)
        b = y
        ends.append(b)
    return ends


@pytest.mark.parametrize("first", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("start,fold_start", [(F(1), False), (F(5), True)], ids=["residue", "basis-conversion"])
def test_doubles(first, start, fold_start):
    # units of 2^50 > p: a product of y is within p / 2 + p |y| 2^-52 (the quotient: wp and the product are rounded), a folded value within
    # p / 2 and the rounding of its quotient; a residue is below p, a converted one within p + 2^52
    stages = ([first] if first else []) + [4, 4, 4]
    ends = steps(start, fold_start, lambda y: F(1, 2) + y / 4, F(1, 2) + F(1, 1 << 40), stages)
    assert max(ends) < 8, [float(e) for e in ends]


@pytest.mark.parametrize("first", [0, 1, 2, 3, 4])
def test_signed_integers(first):
    # units of 2^60: a product of x is within 1 + (1 + |x| / 8) 5 / 16, a folded value within 1/2 and 8 d / 2^60, d < 2^26
    stages = ([first] if first else []) + [4, 4, 4]
    ends = steps(F(114, 100), False, lambda y: 1 + (1 + y / 8) * F(5, 16), F(1, 2) + F(1, 1 << 30), stages)
    assert max(ends) < F(15, 2), [float(e) for e in ends]
