"""The quadrature's sum over its first 36 nodes (GL_SUM in
csrc/ionize_internal.hpp) against all 64, in 80 bits: the rest stays below
2^-60 of the sum for every kT / p and every subshell correction b, c (bound in
the source: 2^-68), far below FP64's last place."""
import os
import re

import numpy as np

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1606_02862_amd", "csrc",
                   "ionize_internal.hpp")


def test_remaining_nodes_are_below_the_last_place():
    n = int(re.search(r"constexpr int GL_SUM = (\d+);", open(SRC).read()).group(1))
    x, w = (a.astype(np.longdouble) for a in np.polynomial.laguerre.laggauss(64))
    assert float((w[n:] * x[n:] ** 2).sum() / (w * x**2).sum()) < 2.0**-67
    for b in (0.0, 0.3, 1.0):
        for c in (0.0, 1e-6, 0.5, 40.0):
            if b == 1.0 and c == 0.0:
                continue  # the rate is zero
            for r in 10.0 ** np.linspace(-12, 12, 97):
                r = np.longdouble(r)
                t = w * np.log1p(x * r) * (b == 0.0 or (1 - b) - b * np.expm1(-c * x * r))
                assert t[n:].sum() < np.longdouble(2.0) ** -60 * t.sum(), (b, c, r)
