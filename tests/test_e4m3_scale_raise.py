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
    assert covered > 9000                                 # 9890 to 33300


SIGNS = np.uint32(0x80808080)


def u32(x):
    return np.asarray(x & 0xffffffff, dtype=np.uint64).astype(np.uint32)


def bytes_of(w):
    return [w >> np.uint32(8 * k) & np.uint32(255) for k in range(4)]


def word_of(parts):
    out = np.uint32(0)
    for k, p in enumerate(parts):
        out = out | np.asarray(p, dtype=np.uint32) << np.uint32(8 * k)
    return out


def perm(hi, lo, select):
    """v_perm_b32 for selectors 0 to 7: byte s of the eight bytes hi:lo."""
    table = bytes_of(np.uint32(lo)) + bytes_of(np.uint32(hi))
    return word_of([np.choose(b.astype(np.int64), table) for b in bytes_of(select)])


def plus(a, b):
    return u32(np.uint64(a) + np.uint64(b))


def minus(a, b):
    return u32(np.uint64(a) + np.uint64(1 << 32) - np.uint64(b))


@pytest.mark.parametrize("spread", [0.02, 0.5, 3.0, 6.0, 40.0])
def test_packed_words_and_tables(spread):
    """The same in the words that the kernel computes with: entries above 60 steps make bytes borrow and carry, and `far`
    has to tell of every such lane; words that are not called uncovered hold the codes of re-encoding raise by raise."""
    rng = np.random.RandomState(int(spread * 100) + 1)
    words = far_chains = 0
    for _ in range(400):
        n = rng.randint(2, 17)
        scales = np.sort(np.exp(rng.uniform(0, spread, n)).astype(F) * F(2.0) ** rng.randint(-50, 30))
        codes = rng.randint(0, 256, (4, 64)).astype(np.int64)
        codes[:, ::5] &= 0x80                             # zeros of both signs
        codes[0, 1::5] &= 0x87                            # subnormals
        want, lo, hi, far, sums = codes & 127, np.uint32(0), np.uint32(0), np.uint32(0), np.zeros(8, dtype=np.int64)
        passed = False
        nan = (want == 127).any(axis=0)
        for s, r in zip(scales, scales[1:]):
            if not r > s:
                continue
            want = raised(np.minimum(want, 126), s, r)
            steps = 0x70 + np.arange(8) - raised(0x70 + np.arange(8), s, r)
            steps = np.where((steps > 60) | (steps < 0), 127, steps)
            sums = sums + steps[(np.arange(8) - sums) & 7]
            passed = passed or bool((sums > 60).any())
            d0, d1 = word_of(steps[:4]), word_of(steps[4:])
            lo, hi = (plus(t, perm(d1, d0, minus(first, t) & np.uint32(0x07070707))) for t, first in ((lo, 0x83828180), (hi, 0x87868584)))
            far = far | plus(lo, 0x43434343) | plus(hi, 0x43434343)
        assert bool(far & SIGNS) == passed                # once set it stays, and it is never set without need
        far_chains += passed
        w = word_of(codes)
        y = minus(w | SIGNS, perm(hi, lo, w & np.uint32(0x07070707)))
        fit = minus(y, 0x08080808)
        low = (y & ~SIGNS) | (w & SIGNS)
        zero = ~plus(w & ~SIGNS, 0x7f7f7f7f) & SIGNS
        same = u32(np.uint64(zero >> np.uint32(7)) * np.uint64(255))
        assert np.array_equal((plus(w & ~SIGNS, 0x01010101) & SIGNS) != 0, nan)
        if passed:
            continue
        again = word_of(want | (codes & 128))
        for out, ok in ((low, (fit & SIGNS) == SIGNS), ((low & ~same) | (w & same), ((fit | zero) & SIGNS) == SIGNS)):
            ok = ok & ~nan
            assert np.array_equal(out[ok], again[ok])
            words += int(ok.sum())
    assert words > 7000 or spread > 3.0
    assert far_chains > 100 or spread <= 3.0


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
