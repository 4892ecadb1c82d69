"""CPU check of the error bound that the l2 exact pass rules rows out with
(chamfer_half_score_bound): the pass's score is emulated exactly as it is
specified -- operands rounded to FP16 (values below 2^-14 to zero), exact
products, float32 accumulation that starts at -|y|^2 / 2 -- with the least
favourable accumulation the bound allows for (every addition truncated), and
its exact error is compared with the bound."""

import math
from fractions import Fraction

import numpy as np
import pytest


def half(v):
    h = np.float16(v)
    return np.where(np.abs(v) < 2.0 ** -14, np.float16(0), h).astype(np.float32)


def truncate(x):
    """x (a Fraction) towards zero to 24 bits."""
    if x == 0:
        return Fraction(0)
    e = math.frexp(float(abs(x)))[1] - 24
    if abs(x) >= Fraction(2) ** (e + 24):
        e += 1
    q = Fraction(2) ** e
    return Fraction(math.trunc(x / q)) * q


def norm(v):
    return math.sqrt(float(np.sum(v.astype(np.float64) ** 2)))


def slots(z, y, d):
    """The products' operands (query side, row side) per slot."""
    zh, yh = half(z), half(y)
    if d > 10:
        return zh, yh, zh, yh
    zm, ym = half(z - zh), half(y - yh)
    return (np.concatenate([zh, zh, zm]), np.concatenate([yh, ym, yh]),
            zh.astype(np.float64) + zm, yh.astype(np.float64) + ym)


@pytest.mark.parametrize("d", [1, 3, 5, 6, 10, 12, 64, 128, 200, 256])
@pytest.mark.parametrize("kind", ["gauss", "same sign", "halfway", "small"])
def test_bound_holds(d, kind):
    import paper_2307_03043_amd as ch
    rng = np.random.default_rng(d)
    worst = 0.0
    for trial in range(6):
        z = rng.standard_normal(d).astype(np.float32) * np.float32(64)
        y = rng.standard_normal(d).astype(np.float32) * np.float32(64)
        if kind == "same sign":  # every partial sum large, every truncation the same way
            z, y = np.abs(z), np.abs(y)
        elif kind == "halfway":  # operands at FP16's rounding boundaries
            z = np.float32(1 + 2.0 ** -11) * np.exp2(rng.integers(0, 8, d)).astype(np.float32)
            y = z[::-1].copy()
        elif kind == "small":    # rounded to zero, or nearly
            z[::2] *= np.float32(2.0 ** -20)
            y[1::2] *= np.float32(2.0 ** -22)
        a, b, zt, yt = slots(z, y, d)
        ze, be = norm(z - zt) * (1 + 1e-6), norm(y - yt) * (1 + 1e-6)
        n2 = np.float32(0)
        for v in y:
            n2 = np.float32(n2 + v * v)
        acc = Fraction(float(-np.float32(0.5) * n2))
        for p, q in zip(a, b):
            acc = truncate(acc + Fraction(float(p)) * Fraction(float(q)))
        exact = sum(Fraction(float(p)) * Fraction(float(q)) for p, q in zip(z, y)) - \
            sum(Fraction(float(q)) ** 2 for q in y) / 2
        E = ch.chamfer_half_score_bound(d, norm(np.asarray(zt)) * (1 + 1e-6), ze,
                                        norm(y) * (1 + 1e-6), be)
        err = abs(float(acc - exact))
        assert err <= E, (trial, err, E)
        worst = max(worst, err / E)
    assert worst > 0.0 or d == 1


def test_bound_arguments():
    import paper_2307_03043_amd as ch
    assert ch.chamfer_half_score_bound(0, 1.0, 0.0, 1.0, 0.0) == -1.0
    assert ch.chamfer_half_score_bound(11, 1.0, 0.0, 1.0, 0.0) == -1.0
    assert ch.chamfer_half_score_bound(257, 1.0, 0.0, 1.0, 0.0) == -1.0
    assert math.isinf(ch.chamfer_half_score_bound(64, 1.0, float("inf"), 1.0, 0.0))
