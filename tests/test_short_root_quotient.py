"""The square root and the quotient that the segmentation's tiles take where no
operand leaves the normal range (sqrt_rn and div_rn of k_pd_tile.hip), step by step
with correctly rounded fused multiply-adds on the host: Newton steps with fused
remainders (P. Markstein, "Computation of elementary functions on the IBM RISC
System/6000 processor", IBM J. Res. Dev. 34, 1990).  The root is correctly rounded
from any reciprocal root within a unit in the last place.  The quotient is from a
correctly rounded reciprocal (Markstein's theorem, with an approximation within a
unit), which the reciprocal instruction and one step give on gfx950 for every
significand (run over all of them there, 153 exponents)."""
import os
import re

import numpy as np
import pytest

F, D = np.float32, np.float64
SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1312_4746_amd", "csrc",
                   "k_pd_tile.hip")


def fma(a, b, c):
    """RN32(a b + c): the product is exact in FP64, its sum with c rounded to odd
    there, so that the rounding to FP32 is the only one that counts."""
    p, c = a.astype(D) * b.astype(D), c.astype(D)
    s = p + c
    t = s - p
    err = (p - (s - t)) + (c - t)
    bits = s.view(np.int64)
    toward = np.where(err == 0, 0, np.where((err > 0) == (s > 0), 1, -1))
    odd = np.where((err != 0) & (bits % 2 == 0), np.where(toward > 0, 1, -1), 0)
    return (bits + odd).view(D).astype(F)


def ulps(x, k):
    return (x.view(np.int32) + np.int32(k)).view(F)


def sqrt_rn(x, r0):
    s, h = x * r0, F(0.5) * r0
    e = fma(-h, s, np.full_like(x, 0.5))
    h = fma(h, e, h)
    s = fma(s, e, s)
    return fma(fma(-s, s, x), h, s)


def div_rn(n, d, y):
    q = n * y
    q = fma(fma(-d, q, n), y, q)
    return q, fma(fma(-d, q, n), y, q)


def mantissas(first, step, binades=1):
    m = np.arange(first, binades << 23, step, dtype=np.int32)
    return (m + np.int32(0x3F800000)).view(F)


def test_the_source_has_these_steps():
    src = re.sub(r"\s+", " ", open(SRC).read())
    for line in ("float s = x * r0, h = 0.5f * r0;", "const float e = fmaf(-h, s, 0.5f);", "h = fmaf(h, e, h);",
                 "s = fmaf(s, e, s);", "return fmaf(fmaf(-s, s, x), h, s);", "y = fmaf(fmaf(-d, y, 1.0f), y, y);",
                 "q = fmaf(fmaf(-d, q, n), y, q);", "return fmaf(fmaf(-d, q, n), y, q);"):
        assert line in src, line


def test_fused_multiply_add_of_the_host():
    from fractions import Fraction
    rng = np.random.default_rng(0)
    a, b, c = (F(2.0) ** rng.integers(-14, 15, 3000).astype(F) * rng.uniform(-2, 2, 3000).astype(F) for _ in range(3))
    c[:1000] = -(a[:1000] * b[:1000])  # cancelling sums
    got = fma(a, b, c)
    for i in range(3000):
        exact = Fraction(float(a[i])) * Fraction(float(b[i])) + Fraction(float(c[i]))
        lo, hi = np.nextafter(got[i], F(-np.inf)), np.nextafter(got[i], F(np.inf))
        d = abs(exact - Fraction(float(got[i])))
        assert d <= abs(exact - Fraction(float(lo))) and d <= abs(exact - Fraction(float(hi)))


@pytest.mark.parametrize("seed", [-1, 0, 1])
def test_root(seed):
    x = mantissas(0, 5, 2)  # [1, 4): a root depends on the parity of the exponent alone
    x = np.concatenate([x, mantissas((2 << 23) - 4096, 1, 2), mantissas(0, 1)[:4096], mantissas(1 << 23, 1, 2)[:4096]])
    r0 = ulps((1.0 / np.sqrt(x.astype(D))).astype(F), seed)
    assert np.array_equal(sqrt_rn(x, r0), np.sqrt(x))


def _quotients(n, d):
    y = (1.0 / d.astype(D)).astype(F)  # (never near a tie: FP64 and then FP32 round as one)
    q, got = div_rn(n, d, y)
    want = n / d
    assert np.array_equal(got, want)
    assert np.all(np.abs(q.view(np.int32) - want.view(np.int32)) <= 1)


@pytest.mark.parametrize("d", [*range(1, 17), 2 - 2.0 ** -23, 1 + 2.0 ** -23])
def test_quotients_of_one_divisor(d):
    n = np.concatenate([mantissas(0, 7), mantissas((1 << 23) - 4096, 1), mantissas(0, 1)[:4096]])
    _quotients(n, np.full_like(n, F(d)))


@pytest.mark.parametrize("seed", range(4))
def test_quotients(seed):
    rng = np.random.default_rng(seed)
    n, d = ((rng.integers(0, 1 << 23, 1 << 20, dtype=np.int32) + np.int32(0x3F800000)).view(F) for _ in range(2))
    _quotients(n, d)
    # near halves between representable quotients: n = (q + half a unit) d, rounded
    q = (1 + rng.random(1 << 20)).astype(F)
    _quotients(((q.astype(D) + 2.0 ** -24) * d).astype(F), d)
