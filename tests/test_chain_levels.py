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

from oracle import rht
from oracle.quantize import quantize

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


def mixed_matrix(m, n):
    """A matrix whose runs of four stages take turns: all of one magnitude, two magnitudes by
    halves of the run, by stages, by blocks of a stage."""
    k = np.arange(n // 16)
    run, stage, block = k // 16 % 4, k // 4 % 4, k % 4
    e = -5 * np.where(run == 1, stage // 2, np.where(run == 2, stage % 2, np.where(run == 3, block % 2, 0)))
    x = np.random.default_rng(m + n).standard_normal((m, n)).astype(np.float32)
    x *= np.exp2(e.repeat(16)).astype(np.float32)
    return (x / np.linalg.norm(x.astype(np.float64))).astype(np.float32)


def operand_levels(q):
    """The chain levels of an NVFP4 record (rows of the product's operand): per 32 rows, the
    largest bound over runs of one, two and four stages."""
    rows, K = q.codes.shape
    nst = -(-K // 64)
    k2 = np.zeros((rows, nst * 64), np.int64)
    k2[:, :K] = K2[q.codes & 7] * np.where(q.codes & 8, -1, 1)
    sc = np.zeros((rows, nst * 4), np.int64)
    sc[:, :K // 16] = q.scales
    words = [[row_word(k2[r, 64 * s:64 * s + 64].reshape(4, 16), [int(c) for c in sc[r, 4 * s:4 * s + 4]])
              for s in range(nst)] for r in range(rows)]
    return [np.array([[max(run_bound([words[r][s] if s < nst else 15 for s in range(g * j, g * j + g)])
                           for r in range(u, min(u + 32, rows))) for j in range(-(-nst // g))]
                      for u in range(0, rows, 32)]) for g in (1, 2, 4)]


def outcomes(levels):
    """{(stage chains, its run of two holds, its run of four holds): stages of unit pairs}."""
    one, two, four = levels
    count = {}
    for s in range(one.shape[1]):
        held = [np.outer(lv[:, s // g], lv[:, s // g]) < LIM for lv, g in ((one, 1), (two, 2), (four, 4))]
        for key in zip(*(h.reshape(-1).tolist() for h in held)):
            count[key] = count.get(key, 0) + 1
    return count


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


@pytest.mark.parametrize("shape", [(272, 1104), (112, 2000), (48, 4240), (16, 32848)])
def test_mixed_matrix_has_every_outcome(shape):
    """The GPU test's matrices reach every kind of stage: none of its bounds holds, its own
    only, its run of two, its run of four (each a twentieth of all stages at least)."""
    q = quantize(mixed_matrix(*shape), 1, rht.step_signs(7, 2), True)
    count = outcomes(operand_levels(q))
    assert set(count) == {(False, False, False), (True, False, False), (True, True, False), (True, True, True)}
    assert min(count.values()) >= sum(count.values()) / 20
