"""The kernels' double-precision exponential (csrc/device_fp64.h), from its source: the polynomial
against the series, and its steps in exactly rounded arithmetic against 40 digits.

The polynomial's own error is to be lost in the roundings: the coefficients', the largest 2^-56 |r|^3 =
5.8e-19, allow it 1e-18, a fiftieth of the last rounding.
A result is rounded once (0.5 units) after a
product with r of a rounded factor (0.35 x 0.5 of the next larger unit, of the result's 0.18 - 0.35)
and carries r's own rounding (0.18 - 0.25): less than one unit in all.
"""
import os
import re
from decimal import Decimal as D
from decimal import localcontext
from fractions import Fraction as F

import numpy as np

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1110_1379_amd", "csrc",
                      "device_fp64.h")
NUMBER = r"-?0x1?\.?[0-9a-f.]*p[+-]?\d+"


def source():
    text = open(HEADER).read()
    body = text[text.index("double exp_(double x)"):]
    body = body[:body.index("\n}")]
    steps = re.findall(r"v_fma_f64 %0, (?:%1, %2|%0, %1), (%\d+|0\.5|1\.0)", body)
    constants = [float.fromhex(v) for v in re.findall(r'"[vs]"\((%s)\)' % NUMBER, body)]
    coefficients = [constants[0]]
    for s in steps:
        coefficients.append(constants[int(s[1:]) - 2] if s[0] == "%" else float(s))
    ln2 = [float.fromhex(v) for v in re.findall(r"__builtin_fma\(k, (%s), [xr]\)" % NUMBER, body)]
    return coefficients, ln2, float(re.search(r"rint\(x \* ([0-9.]+)\)", body).group(1))


def test_polynomial_is_below_the_roundings():
    coefficients, ln2, _ = source()
    assert len(ln2) == 2 and coefficients[-3:] == [0.5, 1.0, 1.0]
    with localcontext() as c:
        c.prec = 50
        assert abs(sum(D(-v) for v in ln2) - D(2).ln()) < D("1e-32")
        a = D(2).ln() / 2
        worst = D(0)
        for i in range(-200, 201):
            r, s = a * i / 200, D(0)
            for v in coefficients:
                s = s * r + D(v)
            worst = max(worst, abs(s / r.exp() - 1))
    assert worst <= D("1e-18"), worst


def test_steps_stay_within_one_unit():
    coefficients, ln2, inv = source()
    fma = lambda x, y, z: float(F(x) * F(y) + F(z))  # noqa: E731
    rng = np.random.default_rng(1)
    worst = 0.0
    with localcontext() as c:
        c.prec = 40
        for x in np.concatenate([rng.uniform(-40, 0, 1500), rng.uniform(-700, 700, 500)]):
            x = float(x)
            k = float(np.rint(x * inv))
            r = fma(k, ln2[1], fma(k, ln2[0], x))
            q = coefficients[0]
            for v in coefficients[1:]:
                q = fma(q, r, v)
            true = D(x).exp() / (D(2) ** int(k))
            worst = max(worst, float(abs(D(q) - true)) / (2.0 ** -53 if true < 1 else 2.0 ** -52))
    assert worst < 1.0, worst
