"""The kernels' division by a divisor known beforehand (`div_by` in csrc/dyn_device.h), its three operations emulated with
whole numbers: every pair of significands of few bits, and at 53 bits those whose quotient lies closest to the midpoint of
two neighbours, where a wrong last bit would show."""
import random

import pytest


def rn(m, p):
    """The whole number m rounded to p significant bits, ties to even."""
    s, m = (-1 if m < 0 else 1), abs(m)
    k = m.bit_length() - p
    if k <= 0:
        return s * m
    q, r = m >> k, m & ((1 << k) - 1)
    h = 1 << (k - 1)
    q += r > h or (r == h and q & 1)
    return s * (q << k)


def quotient(x, y, p):
    """RN(x / y) in units of 2^-(3p); the sticky bit stands below every rounding position."""
    q, r = divmod(x << (3 * p), y)
    return rn((q << 1) | (r != 0), p) >> 1


def div_by(x, y, p):
    z = quotient(1 << p, y, p)                    # RN(1 / y) in units of 2^-(4p)
    one = 4 * p
    q0 = rn(x * z, p)                             # units of 2^-(4p)
    e0 = rn((x << one) - y * q0, p)
    q = rn((q0 << one) + e0 * z, p)               # units of 2^-(8p)
    return q, 5 * p                               # q / 2^(5p) is in units of 2^-(3p)


def same(x, y, p):
    q, shift = div_by(x, y, p)
    return q == quotient(x, y, p) << shift


@pytest.mark.parametrize("p", [3, 4, 5, 6, 7, 8, 9, 10])
def test_every_pair_of_few_bits(p):
    r = range(1 << (p - 1), 1 << p)
    assert all(same(x, y, p) for y in r for x in r)


@pytest.mark.parametrize("below", [0, 1 << 20, 1 << 40, 1 << 52])
def test_quotients_next_to_a_midpoint(below):
    """x 2^54 = m y + k with m odd: x / y is k 2^-106 / y from a midpoint.  Divisors at the upper end of the binade, where the
    reciprocal's error weighs most, and all over it."""
    p, rng, seen = 53, random.Random(5), 0
    for i in range(400):
        y = (1 << 53) - 1 - 2 * i if below == 0 else (1 << 53) - 1 - 2 * rng.randrange(below // 2)
        inv = pow(y, -1, 1 << 54)
        for k in (1, -1, 2, -2, 3, -3, 4, -4, 5, -5, 6, -6):
            m = -k * inv % (1 << 54)
            x = (m * y + k) >> 54
            if m & 1 and m > 1 << 53 and 1 << 52 <= x < y:
                seen += 1
                assert same(x, y, p), (x, y, k)
        inv = pow(y, -1, 1 << 53)                 # x >= y: the quotient's midpoints are twice as far apart
        for k in (1, -1, 3, -3):
            m = -k * inv % (1 << 53)
            m += 1 << 53
            x = (m * y + k) >> 53
            if m & 1 and y <= x < 1 << 53:
                seen += 1
                assert same(x, y, p), (x, y, k)
        for x in (y - 2, (1 << 53) - 1, (1 << 53) - 2, 1 << 52, rng.randrange(1 << 52, 1 << 53)):
            assert same(x, y, p), (x, y)
    assert seen > 200
