"""The rate quadrature's sum (csrc/ionize_internal.hpp), run on the CPU, against
80-bit arithmetic: with the table logarithm and 36 of the 64 nodes it is no
further from its value than one chain over all nodes with the library's log1p,
in the mean and in the square mean, over every kT / p the rates meet."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")


@pytest.fixture(scope="module")
def sums(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rate_sum") / "librate_sum.so")
    subprocess.check_call(["hipcc", "-O2", "-std=c++17", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", so,
                           os.path.join(HERE, "rate_sum_host.hip")], stderr=subprocess.DEVNULL)
    lib = C.CDLL(so)
    rule = np.concatenate(np.polynomial.laguerre.laggauss(64))

    def run(r, b, c):
        out = np.empty((2, r.size))
        ptr = lambda a: a.ctypes.data_as(C.c_void_p)  # noqa: E731
        lib.rsh_sum(C.c_int64(r.size), ptr(r), ptr(b), ptr(c), ptr(rule), ptr(out[0]), ptr(out[1]))
        x, w = rule[:64].astype(np.longdouble), rule[64:].astype(np.longdouble)
        ref = np.zeros(r.size, dtype=np.longdouble)
        for k in range(64):
            xr = x[k] * r
            ref += w[k] * np.log1p(xr) * (1 - b * np.exp(-c * xr))
        return out[0], out[1], ref
    return run


@pytest.mark.parametrize("corrected", [False, True])
@pytest.mark.parametrize("lo,hi", [(-8, -3), (-3, 0), (0, 3), (3, 8)])
def test_no_further_from_the_value_than_a_plain_sum(sums, lo, hi, corrected):
    g = np.random.default_rng(11)
    n = 40_000
    r = 10.0 ** g.uniform(lo, hi, n)
    # b up to 1/2: from there on 1 - b e^{-c x r} itself cancels in either sum
    b = g.uniform(0.05, 0.5, n) if corrected else np.zeros(n)
    c = 10.0 ** g.uniform(-2, 1, n)
    got, plain, ref = sums(r, b, c)
    e, p = (np.abs((v - ref) / ref).astype(np.float64) for v in (got, plain))
    print(lo, hi, corrected, e.mean() * 2**53, p.mean() * 2**53, flush=True)
    assert e.mean() <= p.mean() and (e**2).mean() <= (p**2).mean() and e.max() <= max(p.max(), 4 * 2.0**-52)
