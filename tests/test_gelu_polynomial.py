"""The polynomial of the GELU epilogue (gemm.hip gelu_erf), read from the
source and evaluated in FP64: v / (1 + 2^(-v q(v^2))) is within the stated
6.7e-8 of v Phi(v) for every v, and no polynomial of its degree fitted the
same way does better by more than float32 rounding of the coefficients."""
import os
import re

import numpy as np
from scipy.optimize import linprog
from scipy.special import log_ndtr, ndtr

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _coefficients():
    text = open(os.path.join(ROOT, "paper_2604_27441_amd", "csrc", "gemm.hip")).read()
    body = text[text.index("float gelu_erf(float v)"):]
    body = body[:body.index("return v *")]
    c = [float(x) for x in re.findall(r"(-?\d\.\d+(?:e[-+]?\d+)?)f", body)]
    assert len(c) == 7
    return c[::-1]   # the source nests from the highest power


def test_error_of_the_gelu_polynomial():
    c = _coefficients()
    v = np.linspace(-40, 40, 4000001)
    with np.errstate(over="ignore"):
        got = v / (1 + np.exp2(-v * np.polyval(c[::-1], v * v)))
    assert np.abs(got - v * ndtr(v)).max() <= 6.75e-8


def test_coefficients_are_the_minimax_fit():
    """Minimise the largest first-order error of v Phi(v), weight
    v^2 Phi (1 - Phi) ln 2, over v in (0, 7]: a linear program."""
    v = np.linspace(1e-3, 7.0, 2001)
    q = (log_ndtr(v) - log_ndtr(-v)) * np.log2(np.e) / v
    w = 1e6 * v * v * ndtr(v) * ndtr(-v) * np.log(2)
    a = np.vander(v * v / 49.0, 7, increasing=True) * w[:, None]
    one = np.ones((v.size, 1))
    res = linprog(np.r_[np.zeros(7), 1.0], A_ub=np.block([[a, -one], [-a, -one]]), b_ub=np.r_[w * q, -w * q],
                  bounds=[(None, None)] * 7 + [(0, None)], method="highs")
    best = res.x[-1] * 1e-6
    ours = np.abs(w * (np.polyval(_coefficients()[::-1], v * v) - q)).max() * 1e-6
    assert ours <= 1.02 * best, (ours, best)
