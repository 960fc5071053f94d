"""Readback of more particles than one staging chunk holds (2,097,152), ids in
random order: every value beside its id, as the host sort has it."""
import numpy as np
import pytest

import workloads
from tests.test_gpu_scratch_failure import _Refusing

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_two_chunks(precision):
    import paper_1606_02862_amd as P
    P.load()
    cfg = workloads.config(0, nx=64, ny=64, nz=64, precision=precision)
    cfg["species"][0]["ppc"] = 9
    alloc = _Refusing(P)
    with P.Pic(cfg, allocator=alloc) as pic:
        n = pic.count(0)
        assert n > 2_097_152 and n % 2_097_152
        p = pic.get_particles(0)
        p["id"] = np.random.default_rng(2).permutation(n).astype(np.int64)
        pic.set_particles(0, p)
        got = pic.get_particles(0)
        alloc.arm(1)
        want = pic.get_particles(0)
        assert alloc.refused == 1
    order = np.argsort(p["id"])
    for k in p:
        assert np.array_equal(got[k], want[k]) and np.array_equal(got[k], p[k][order]), k
