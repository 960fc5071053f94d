"""The readback's page backing (csrc/page_touch.hpp), run on the CPU: the output
arrays keep what they hold, to the byte, since the call may still fail; bytes
beside them are not touched either; and fresh pages are in place afterwards."""
import ctypes as C
import os
import resource
import subprocess

import numpy as np
import pytest

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")


@pytest.fixture(scope="module")
def touch(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("page_touch") / "libpage_touch.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", "-pthread", "-o", so,
                           os.path.join(HERE, "page_touch_host.cpp")])
    lib = C.CDLL(so)

    def run(spans):
        p = (C.c_void_p * 9)(*[a for a, _ in spans])
        n = (C.c_size_t * 9)(*[b for _, b in spans])
        return lib.pth_touch(p, n)
    return run


@pytest.mark.parametrize("size", [0, 1, 4096, 3_000_001])
def test_contents_stay(touch, size):
    g = np.random.default_rng(3)
    arrays = [g.integers(1, 255, size + 64, dtype=np.uint8) for _ in range(8)]
    before = [a.copy() for a in arrays]
    touch([(a.ctypes.data + 7 * i % 64, size) for i, a in enumerate(arrays)] + [(None, 0)])  # the last: no zstate array
    for a, b in zip(arrays, before):
        assert np.array_equal(a, b)


def test_fresh_pages_are_backed(touch):
    arrays = [np.zeros(16 << 20, dtype=np.uint8) for _ in range(2)]
    assert touch([(a.ctypes.data, a.nbytes) for a in arrays] + [(None, 0)] * 7) > 0
    before = resource.getrusage(resource.RUSAGE_SELF).ru_minflt
    for a in arrays:
        a[::4096] = 1
    assert resource.getrusage(resource.RUSAGE_SELF).ru_minflt - before < 100  # of 8192 pages
