"""The rate quadrature's ln(1 + y) (csrc/rate_log.hpp), run on the CPU, against
80-bit logarithms.

Bound: the table constant, the polynomial (2^-59 of t) and the final two
roundings leave at most 1.5 units in the last place (2^-53 each of the
result, plus 2^-53 of the larger of the terms added), for every y in range.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")


@pytest.fixture(scope="module")
def log1p(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rate_log") / "librate_log.so")
    subprocess.check_call(["hipcc", "-O2", "-std=c++17", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", so,
                           os.path.join(HERE, "rate_log_host.hip")], stderr=subprocess.DEVNULL)
    lib = ctypes.CDLL(so)

    def run(y):
        y = np.ascontiguousarray(y, dtype=np.float64)
        out = np.empty_like(y)
        ptr = lambda a: a.ctypes.data_as(ctypes.POINTER(ctypes.c_double))  # noqa: E731
        lib.rlh_log1p(ctypes.c_int64(y.size), ptr(y), ptr(out))
        return out
    return run


@pytest.mark.parametrize("lo,hi", [(1e-320, 1e-17), (1e-17, 1e-2), (1e-2, 1.0), (1.0, 1e4), (1e4, 1e17), (1e17, 1e300)])
def test_log1p_matches_80_bits(log1p, lo, hi):
    g = np.random.default_rng(5)
    y = np.concatenate([10.0 ** g.uniform(np.log10(lo), np.log10(hi), 400_000), [lo, hi]])
    y = y[(y >= lo) & (y <= hi)]
    want = np.log1p(y.astype(np.longdouble))
    err = np.abs(log1p(y) - want) / np.spacing(want.astype(np.float64))
    assert err.max() <= 1.5, (y[err.argmax()], err.max())


def test_log1p_at_table_edges(log1p):
    """The ends of every table interval at several exponents, and zero."""
    m = 1.0 + np.arange(129) / 128.0
    u = np.concatenate([np.ldexp(np.concatenate([m, np.nextafter(m, 0), np.nextafter(m, 4)]), e) for e in (0, 1, 2, 7, 30, 60)])
    y = np.concatenate([u[u >= 1.0] - 1.0, [0.0]])
    want = np.log1p(y.astype(np.longdouble))
    err = np.abs(log1p(y) - want) / np.spacing(want.astype(np.float64))
    assert err.max() <= 1.5
    assert log1p([0.0])[0] == 0.0
