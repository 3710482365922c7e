"""The chain bounds of the NVFP4 products over runs of stages, as the kernels form them.

Each 64-element stage of a row is one word: T = sum n2_b 4^(E_b) in binary32 rounded up
to 28 bits, and in the low four bits the smallest unit exponent e_b = E_b + (trailing
zeros of the scale's significand), at most 15.  A run of stages sums the words' T, takes
their smallest e and multiplies by 4^(-e).  Claim: if the bounds of two rows multiply to
less than 2^48 (1 - 2^-16), every product of the run is an integer multiple of
u = 2^(ea + eb - 22) and the sum of their magnitudes is at most 2^24 u.  Checked with
integer arithmetic on random rows, power-of-two significands and zero blocks.
"""
from fractions import Fraction
import math

import numpy as np
import pytest

K2 = np.array([0, 1, 2, 3, 4, 6, 8, 12])
LIM = 2.0 ** 48 * (1 - 2.0 ** -16)


def parts(code):
    ef, mf = (code >> 3) & 15, code & 7
    return (8 + mf, ef) if ef else (mf, 1)


def unit_exp(code):
    m, e = parts(code)
    return 15 if m == 0 else min(e + (m & -m).bit_length() - 1, 15)


def row_word(k2, codes):
    t = [np.float32(float(int(np.sum(k2[b] ** 2)) * parts(c)[0] ** 2 * 4 ** parts(c)[1])) for b, c in enumerate(codes)]
    s = np.float32(np.float32(t[0] + t[1]) + np.float32(t[2] + t[3]))
    return ((int(s.view(np.uint32)) + 31) & ~15) | min(unit_exp(c) for c in codes)


def run_bound(words):
    t = [np.uint32(w & ~15).view(np.float32) for w in words]
    while len(t) > 1:
        t = [np.float32(t[i] + t[i + 1]) for i in range(0, len(t), 2)]
    rho = float(t[0]) * 4.0 ** -min(w & 15 for w in words)
    return float(np.float32(np.float32(rho) * np.float32(1 + 2.0 ** -20)))


def make_row(rng, stages, lo, hi, kind):
    k2 = rng.choice(K2, size=(stages, 4, 16)) * rng.choice([-1, 1], size=(stages, 4, 16))
    e = rng.integers(lo, hi + 1, size=(stages, 4))
    m = rng.integers(0, 8, size=(stages, 4)) if kind != "pow2" else rng.choice([0, 4], size=(stages, 4))
    codes = (e << 3) | m
    if kind == "zeros":
        codes[rng.random((stages, 4)) < 0.3] = 0
    return k2, codes


@pytest.mark.parametrize("stages", [1, 2, 4])
@pytest.mark.parametrize("kind", ["plain", "pow2", "zeros"])
def test_run_bound_covers_every_partial_sum(stages, kind):
    rng = np.random.default_rng(11 * stages + len(kind))
    held = 0
    for trial in range(150):
        spread = int(rng.integers(0, 6))
        lo = int(rng.integers(0, 9))
        ka, ca = make_row(rng, stages, lo, min(lo + spread, 15), kind)
        kb, cb = make_row(rng, stages, lo, min(lo + spread, 15), kind)
        if trial % 10 == 0:
            kb, cb = ka, ca                       # Cauchy-Schwarz with equality
        wa = [row_word(ka[s], [int(c) for c in ca[s]]) for s in range(stages)]
        wb = [row_word(kb[s], [int(c) for c in cb[s]]) for s in range(stages)]
        if run_bound(wa) * run_bound(wb) >= LIM:
            continue
        held += 1
        unit = Fraction(2) ** (min(w & 15 for w in wa) + min(w & 15 for w in wb) - 22)
        total = Fraction(0)
        for s in range(stages):
            for b in range(4):
                (ma, ea), (mb, eb) = parts(int(ca[s, b])), parts(int(cb[s, b]))
                f = Fraction(ma * mb) * Fraction(2) ** (ea + eb - 22)
                for x, y in zip(ka[s, b], kb[s, b]):
                    p = int(x) * int(y) * f
                    assert (p / unit).denominator == 1
                    total += abs(p)
        assert total <= unit * 2 ** 24
    assert held > 20


def test_rounding_up():
    """The word's T is never below the exact sum, and exceeds it by at most 47 ulps."""
    rng = np.random.default_rng(3)
    for _ in range(300):
        k2, codes = make_row(rng, 1, 1, 15, "plain")
        exact = sum(int(np.sum(k2[0, b] ** 2)) * parts(int(c))[0] ** 2 * 4 ** parts(int(c))[1]
                    for b, c in enumerate(codes[0]))
        t = float(np.uint32(row_word(k2[0], [int(c) for c in codes[0]]) & ~15).view(np.float32))
        assert exact <= t <= exact + 47 * 2.0 ** (math.frexp(float(exact))[1] - 23)
