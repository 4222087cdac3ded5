"""Host-side check of the arithmetic shortcut the quantising kernels take: with r = fl(1 / s), the sums of 2^23 + 2^22 + offset and the
exact products x * r (1 - 2^-21) and x * r (1 + 2^-21), each rounded once to single precision, carry rne(x / s) + offset in
their lowest byte wherever the two agree; where they differ the kernels divide.  Fused multiply-adds are taken in exact integer
arithmetic here; the kernels themselves are compared with the oracle, bit for bit, in the GPU tests."""
from fractions import Fraction

import numpy as np
import pytest

import synth_inputs as S

F = np.float32


def _fused_sum(x, r, magic):
    """fl(x * r + magic), exact product, one rounding: x fp16, r single, magic with a unit in the last place of 1 (|x * r| < 2^22,
    so the sum is an integer: round half to even of the exact value)."""
    p = x.astype(np.float64) * np.float64(r)   # 11 + 24 bits: exact in double
    return np.rint(p) + np.float64(magic)      # rint: half to even; magic is even


def _codes(x, s, offset):
    """(codes where the two sums agree, mask of agreement), as the kernels compute them."""
    r = F(1.0) / s
    r_lo, r_hi = r * F(1.0 - 2.0 ** -21), r * F(1.0 + 2.0 ** -21)
    magic = 12582912.0 + offset
    lo, hi = _fused_sum(x, r_lo, magic), _fused_sum(x, r_hi, magic)
    bits = lo.astype(F).view(np.uint32)
    return (bits & 0xFF).astype(np.int64) - offset, lo == hi


def _check(x, s, offset):
    x = x.astype(np.float16)
    code, agree = _codes(x, s, offset)
    true = np.rint(x.astype(F) / s)
    assert np.array_equal(code[agree], true[agree])
    return int((~agree).sum()), x.size


def test_fused_sum_is_the_rounded_exact_value():
    rng = np.random.default_rng(1)
    x = (rng.standard_normal(200) * 10.0 ** rng.uniform(-4, 2, 200)).astype(np.float16)
    for offset in (8, 128):
        for r in (F(0.37), F(12.7), F(1.0) / F(3.0)):
            got = _fused_sum(x, r, 12582912.0 + offset)
            for v, g in zip(x, got):
                exact = Fraction(float(v)) * Fraction(float(r))
                n = exact.numerator // exact.denominator
                rest = exact - n
                n += 1 if rest > Fraction(1, 2) or (rest == Fraction(1, 2) and n % 2) else 0
                assert g == 12582912 + offset + n and F(g) == g


@pytest.mark.parametrize("hi,offset", [(127, 128), (7, 8)])
def test_agreeing_sums_give_the_quotients_code(hi, offset):
    apart = total = 0
    for seed in range(6):
        x = S.activations_outlier(64, 4096, seed=900 + seed).astype(np.float16)
        for row in x:
            amax = F(np.abs(row.astype(F)).max())
            u, n = _check(row, amax / F(hi), offset)
            apart += u
            total += n
    # the products lie |x / s| * 2^-20 apart, so that often a value's boundary falls between them: one in 8000 at |x / s| = 127
    assert apart <= total * hi * 2.0 ** -20 * 2 + 8


@pytest.mark.parametrize("hi,offset", [(127, 128), (7, 8)])
def test_values_next_to_rounding_boundaries(hi, offset):
    rng = np.random.default_rng(5)
    apart = 0
    for _ in range(200):
        amax = F(np.float16(rng.uniform(0.5, 300.0)))
        s = amax / F(hi)
        k = rng.integers(-hi, hi, size=512)
        # fp16 values as close as fp16 allows to (k + 1/2) s, on both sides
        x = ((k + 0.5) * float(s)).astype(np.float16)
        near = np.concatenate([x, np.nextafter(x, np.float16(np.inf)), np.nextafter(x, np.float16(-np.inf))])
        near = near[np.abs(near.astype(F)) <= amax]
        apart += _check(near, s, offset)[0]
    assert apart > 0  # the division is needed here and there
