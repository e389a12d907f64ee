"""Re-encoding e4m3 codes under a raised scale by a table of eight entries, and quotients without a division: what the
chunk append rests on.

encode(decode(c) * s / r) with every operation rounded to fp32, s < r: as long as code and outcome are normal numbers,
the code falls by a number of steps that its three mantissa bits decide, two raises in a row are one table, and the
outcome shows (a result below the smallest normal code) where that does not hold."""
from fractions import Fraction

import numpy as np
import pytest

F = np.float32


def decode(code):
    e, m = code >> 3, code & 7
    return np.where(e > 0, np.ldexp(F(1) + m.astype(F) / F(8), e - 7), np.ldexp(m.astype(F) / F(8), -6)).astype(F)


MAGNITUDES = decode(np.arange(127)).astype(np.float64)


def encode(y):
    """Nearest of the 127 finite magnitudes, ties to the even code, saturating."""
    y = np.minimum(y.astype(np.float64), 448.0)
    hi = np.clip(np.searchsorted(MAGNITUDES, y), 1, 126)
    below, above = y - MAGNITUDES[hi - 1], MAGNITUDES[hi] - y
    return np.where((below < above) | ((below == above) & ((hi - 1) % 2 == 0)), hi - 1, hi)


def raised(codes, s, r):
    return encode(((decode(codes) * s).astype(F) / r).astype(F))


@pytest.mark.parametrize("spread", [0.02, 0.5, 3.0, 6.0])
def test_table_of_raises(spread):
    rng = np.random.RandomState(int(spread * 100))
    codes = np.arange(127)
    covered = 0
    for _ in range(300):
        scales = np.sort(np.exp(rng.uniform(-1, spread, 6)).astype(F) * F(2.0) ** rng.randint(-60, 60))
        want, low, far = codes, np.zeros(8, dtype=np.int64), False
        for s, r in zip(scales, scales[1:]):
            if not r > s:
                continue
            want = raised(want, s, r)
            steps = 0x70 + np.arange(8) - raised(0x70 + np.arange(8), s, r)
            low = low + np.where(steps > 60, 127, steps)[(np.arange(8) - low) & 7]
            far = far or bool((low > 60).any())
        if far:
            continue
        got = codes - low[codes & 7]
        ok = got >= 8                                     # both normal: the code before is never the smaller one
        assert np.array_equal(got[ok], want[ok])
        assert (want[~ok] <= 8).all()                     # nothing that stays normal goes unseen
        covered += int(ok.sum())
    assert covered > 300


def exponent(x):
    e = abs(x.numerator).bit_length() - x.denominator.bit_length()
    return e - (Fraction(2) ** e > abs(x))


def rounded(x):
    """A rational to the nearest number of 24 binary digits, ties to even."""
    unit = Fraction(2) ** (exponent(x) - 23) if x else 1
    return round(x / unit) * unit


def test_corrected_quotients_of_bf16_over_scale():
    """v / s for every pair of bf16 mantissas v and a with s = a / 448 rounded: the quotient by a reciprocal that may be a
    unit off either way, corrected once by its exact remainder, is the correctly rounded one."""
    for a in range(128, 256):
        s = rounded(Fraction(a, 448))
        r = rounded(1 / s)
        unit = Fraction(2) ** (exponent(r) - 23)
        for v in range(128, 256):
            want = rounded(v / s)
            for near in (r - unit, r, r + unit):
                q = rounded(v * near)
                assert rounded(rounded(q * s - v) * -near + q) == want, (a, v)
