"""The digits of fp32 logits (score_fixed.h) in exact integers: what their test lets pass is as good as an fp32 rounding.

A row is a fixed-point vector of 46 bits and a sign below 2^e, its largest element's next power of two, in six balanced
base-256 digits; products of digits beyond the seventh level are left out, and the sum is cut to whole units of 2^(E - 51),
E = ex + ey.  A dot product below 2^-17 2^E, or below 2^-12 2^E where either row has an element with bits below its digits,
is formed in fp64 instead.
"""
import random
from fractions import Fraction

import pytest

DIGITS, LEVELS = 6, 7
LEAST, LEAST_CUT = Fraction(1, 2 ** 17), Fraction(1, 2 ** 12)
# Of what passes, relative: the levels left out are at most 4 * 2^14 * 2^24 + 3 * 2^14 * 2^16 of 2^92 per element, the cut to
# whole units two of them; an element cut off is off by 2^-47 of its row and meets one below 2^e of the other.
D = 128
LEFT_OUT = Fraction(D * (4 * 2 ** 38 + 3 * 2 ** 30 + 2 * 2 ** 22 + 2 ** 14), 2 ** 92) + Fraction(2, 2 ** 51)
BOUND = LEFT_OUT / LEAST
BOUND_CUT = (2 * Fraction(D, 2 ** 47) * (1 + Fraction(1, 2 ** 47)) + LEFT_OUT) / LEAST_CUT


def fp32(x):
    """Nearest number of 24 significant bits (no subnormals here)."""
    x = Fraction(x)
    if x == 0:
        return x
    e = exponent([x])
    return round(x * Fraction(2) ** (24 - e)) / Fraction(2) ** (24 - e)


def exponent(row):
    """e with max |x| < 2^e, and no smaller one."""
    m = max(abs(x) for x in row)
    e = m.numerator.bit_length() - m.denominator.bit_length()
    return e + 1 if m >= Fraction(2) ** e else e


def digits(row):
    """(e, digits per element from the highest, whether an element was cut)."""
    e = exponent(row)
    scaled = [x * Fraction(2) ** (8 * DIGITS - 2 - e) for x in row]
    out = []
    for x in scaled:
        n, d = round(x), []                                  # (to even, as the sum with 1.5 * 2^52)
        for _ in range(DIGITS - 1):
            low = (n + 128) % 256 - 128
            d.append(low)
            n = (n - low) >> 8
        assert abs(n) <= 64
        out.append([n] + d[::-1])
    return e, out, any(x.denominator != 1 for x in scaled)


def dot(x, y):
    """(dot product as the digits give it, whether it passes)."""
    ex, dx, cut_x = digits(x)
    ey, dy, cut_y = digits(y)
    level = [sum(a[i] * b[t - i] for a, b in zip(dx, dy) for i in range(max(0, t - 5), min(t, 5) + 1)) for t in range(LEVELS)]
    assert all(abs(s) < 2 ** 31 for s in level)
    hi, mid = (level[0] << 8) + level[1], (level[2] << 8) + level[3]
    lo = (level[4] << 7) + ((level[5] + (level[6] >> 8)) >> 1)
    units = (hi * 65536 + mid) * 32768 + lo                  # of 2^(E - 51), each step exact in fp64
    assert max(abs(hi * 65536 + mid), abs(units)) < 2 ** 53
    return units * Fraction(2) ** (ex + ey - 51), abs(Fraction(units, 2 ** 51)) >= (LEAST_CUT if cut_x or cut_y else LEAST)


def normal(rng, d, scale):
    return [fp32(rng.gauss(0, 1) * s) for s in scale(rng, d)]


BELOW_ONE = 1 - Fraction(1, 2 ** 24)
TINY = Fraction(1, 2 ** 24) * (Fraction(5, 4) + Fraction(1, 2 ** 23))            # half a unit of the 46 bits


def built(d, big_x, big_y):
    """x has its largest element at the first `big_x` places, y at the last `big_y`, and elements that are cut, all the same way,
    where the other has its largest."""
    x = [BELOW_ONE if i < big_x else TINY for i in range(d)]
    y = [(BELOW_ONE if i >= d - big_y else TINY if i < big_x else Fraction(0)) for i in range(d)]
    return x, y


def check(x, y):
    got, held = dot(x, y)
    want = sum(a * b for a, b in zip(x, y))
    if held:
        cut = digits(x)[2] or digits(y)[2]
        assert abs(got - want) <= (BOUND_CUT if cut else BOUND) * abs(got)
    return held, abs(got - want) / abs(want)


def test_bounds():
    assert BOUND < Fraction(1, 2 ** 27) and BOUND_CUT < Fraction(17, 16) / 2 ** 27


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("big", [(1, "rest"), ("half", "half"), ("rest", 1)])
def test_rows_built_against_the_digits(d, big):
    count = {1: 1, "half": d // 2, "rest": d - 1}
    x, y = built(d, count[big[0]], count[big[1]])
    held, error = check(x, y)
    assert digits(x)[2] and not held                         # ...so that it goes to fp64: the digits are off by three roundings
    assert error > Fraction(1, 2 ** 24)


def test_rows_built_against_the_levels():
    """Digits of 128 wherever a level is left out, on rows that the digits hold: the largest error of those."""
    x = fp32(Fraction(sum(127 * 256 ** i for i in range(5)) + 63 * 256 ** 5, 2 ** 46))
    for low in (127 * 257, 127 * 65793, 128 * 65793):
        check([x] + [fp32(Fraction(low, 2 ** 46))] * (D - 1), [x] + [fp32(Fraction(low, 2 ** 46))] * (D - 1))
        check([x / 4] + [fp32(Fraction(low, 2 ** 46))] * (D - 1), [x / 4] * (D - 1) + [x])


SCALES = {
    "normal": lambda rng, d: [1] * d,
    "channels_8": lambda rng, d: [8 if i < 4 else 1 for i in range(d)],
    "binades_20": lambda rng, d: [2.0 ** rng.uniform(-20, 0) for _ in range(d)],
    "binades_30": lambda rng, d: [2.0 ** rng.uniform(-30, 0) for _ in range(d)],
    "channel_2^24": lambda rng, d: [2.0 ** 24 if i == 5 else 1 for i in range(d)],
    "channel_2^-24": lambda rng, d: [2.0 ** -24 if i == 5 else 1 for i in range(d)],
}


@pytest.mark.parametrize("y", SCALES)
@pytest.mark.parametrize("x", SCALES)
def test_random_rows(x, y):
    rng = random.Random("%s/%s" % (x, y))
    for _ in range(20):
        d = rng.choice((64, 128))
        check(normal(rng, d, SCALES[x]), normal(rng, d, SCALES[y]))
