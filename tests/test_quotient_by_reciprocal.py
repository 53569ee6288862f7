"""The sampler's quotient e / z from the rounded reciprocal of z and two residual
corrections must be the correctly rounded one for every e in [2^-80, 1] and z in
[1, 16384] (the softmax's terms and their sum). The five operations are run
here in exact rational arithmetic, each rounded once to binary32."""
from fractions import Fraction

import numpy as np
import pytest


def _rn(x: Fraction) -> Fraction:
    """x rounded to binary32 (normal range), ties to even."""
    if x == 0:
        return x
    n, d = abs(x.numerator), x.denominator
    e = n.bit_length() - d.bit_length()
    if Fraction(n, d) < Fraction(2) ** e:
        e -= 1
    ulp = Fraction(2) ** (e - 23)
    q = Fraction(n, d) / ulp
    k = q.numerator // q.denominator
    rest = q - k
    if rest > Fraction(1, 2) or (rest == Fraction(1, 2) and k & 1):
        k += 1
    return (k * ulp) * (1 if x > 0 else -1)


def _quotient(e: Fraction, z: Fraction) -> Fraction:
    r = _rn(1 / z)
    q = _rn(e * r)
    for _ in range(2):
        rem = _rn(e - q * z)      # one fused operation each
        q = _rn(q + rem * r)
    return q


def _cases(kind, n, rng):
    if kind == "random":
        e = np.exp2(rng.uniform(-80, 0, n)).astype(np.float32)
        z = np.exp2(rng.uniform(0, 14, n)).astype(np.float32)
    elif kind == "mantissa edges":       # significands next to powers of two
        ulps = rng.integers(-4, 5, (2, n)).astype(np.int32)
        e = (np.exp2(rng.integers(-79, 0, n)).astype(np.float32).view(np.int32) + ulps[0]).view(np.float32)
        z = (np.exp2(rng.integers(1, 14, n)).astype(np.float32).view(np.int32) + ulps[1]).view(np.float32)
    else:                                # quotients next to the middle of two floats
        z = np.exp2(rng.uniform(0, 14, n)).astype(np.float32)
        q = np.exp2(rng.uniform(-70, -14, n)).astype(np.float32)
        mid = q.astype(np.float64) * (1 + 2.0 ** -24)
        e = (mid * z).astype(np.float32)
    return np.clip(e, np.float32(2.0 ** -80), np.float32(1)), np.clip(z, np.float32(1), np.float32(16384))


@pytest.mark.parametrize("kind", ["random", "mantissa edges", "midpoints"])
def test_corrected_quotient_is_correctly_rounded(kind):
    e, z = _cases(kind, 4000, np.random.default_rng(11))
    want = e / z
    for a, b, w in zip(e, z, want):
        assert _quotient(Fraction(float(a)), Fraction(float(b))) == Fraction(float(w)), (a, b)
