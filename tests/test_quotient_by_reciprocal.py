"""The sampler's quotient e / z from the rounded reciprocal of z and two residual
corrections must be the correctly rounded one for every e in [2^-80, 1] and z in
[1, 16384] (the softmax's terms and their sum). The five operations are run
here in exact rational arithmetic, each rounded once to binary32; the kernel's
own quotients are compared with its divisions on the GPU."""
from fractions import Fraction

import numpy as np
import pytest


def _rn(x: Fraction) -> Fraction:
    """x rounded to binary32 (below its largest value), ties to even."""
    if x == 0:
        return x
    n, d = abs(x.numerator), x.denominator
    e = n.bit_length() - d.bit_length()
    if Fraction(n, d) < Fraction(2) ** e:
        e -= 1
    ulp = Fraction(2) ** max(e - 23, -149)
    q = Fraction(n, d) / ulp
    k = q.numerator // q.denominator
    rest = q - k
    if rest > Fraction(1, 2) or (rest == Fraction(1, 2) and k & 1):
        k += 1
    return (k * ulp) * (1 if x > 0 else -1)


def _quotient(e: Fraction, z: Fraction, corrections: int = 2) -> Fraction:
    r = _rn(1 / z)
    q = _rn(e * r)
    for _ in range(corrections):
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


def _softmax_terms(V, spread, rng):
    """Logits from 0 down to -spread, and exp of them, in the GPU test's rows."""
    x = (-spread * rng.random(V)).astype(np.float32)
    x[rng.integers(0, V)] = 0.0
    x[rng.integers(0, V)] = -spread
    return x, np.exp(x.astype(np.float64)).astype(np.float32)


def _wrong(spread, corrections, n=4000):
    """How many of n quotients of such a row the corrections leave wrong."""
    _, e = _softmax_terms(n, spread, np.random.default_rng(13))
    z = np.float32(e.sum(dtype=np.float32))
    want = e / z
    return sum(_quotient(Fraction(float(a)), Fraction(float(z)), corrections) != Fraction(float(w))
               for a, w in zip(e, want))


def test_the_rows_tell_missing_corrections_and_a_missing_guard():
    """The first correction already leaves no sample wrong (the second is what the
    proof needs), so rows can tell only that there is none."""
    assert _wrong(10.0, 2) == _wrong(54.0, 2) == 0
    assert _wrong(10.0, 0) > 100
    assert _wrong(87.0, 2) > 0              # remainders below the smallest subnormal


@pytest.mark.gpu
@pytest.mark.parametrize("V", [60, 2052, 16384])
def test_kernel_quotients_equal_its_divisions(V):
    """An entry at -200 below the largest has exp 0. Dropped by top-k it leaves the
    row's range to the reciprocal (up to a spread of 55); kept it forces the
    division, with the same sum. So every p must come out the same bit for bit."""
    torch = pytest.importorskip("torch")
    import paper_2608_18183_amd as P
    rng = np.random.default_rng(V)
    spreads = [0.01, 1.0, 3.0, 10.0, 30.0, 50.0, 54.0, 54.9, 55.1, 60.0, 75.0, 87.0]
    x = np.stack([_softmax_terms(V, s, rng)[0] for s in spreads for _ in range(4)])
    for row in x:
        k = rng.integers(1, V - 1)
        while row[k] == 0.0 or row[k] == row.min():
            k = rng.integers(1, V - 1)
        row[k] = -200.0
    n = len(x)
    dev = torch.from_numpy(x).cuda()
    one, pos = torch.ones(n, device="cuda"), torch.ones(n, dtype=torch.int32, device="cuda")
    by_reciprocal = P.hbsjd_transform_rows(dev, one, pos, top_k=V - 1)[0].cpu().numpy()
    by_division = P.hbsjd_transform_rows(dev, one, pos, top_k=0)[0].cpu().numpy()
    assert np.all(by_division[x == -200.0] == 0) and np.all(by_division[x > -88.0] > 0)
    assert np.array_equal(by_reciprocal.view(np.int32), by_division.view(np.int32))
