"""Device memory refused in the middle of a run: the call that asked for it
reports it or does without, and the calls after it are unaffected.  A refused
hipMalloc stays behind as the runtime's last error, which the launches that
follow must not take for their own."""
import ctypes as C

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    import paper_1606_02862_amd as pkg
    pkg.load()
    return pkg


class _Refusing:
    """torch device memory; while armed, request number `at` (and every later
    one) asks hipMalloc for more than any card holds and hands on its failure."""

    def __init__(self, P):
        from paper_1606_02862_amd import _capi as A
        self.lib, self.live, self.at, self.calls, self.refused = P.load(), {}, None, 0, 0
        self._alloc = A.ALLOC_FN(self._do_alloc)
        self._free = A.FREE_FN(self._do_free)
        self.struct = A.AllocT(self._alloc, self._free, None)

    def arm(self, at):
        self.at, self.calls, self.refused = at, 0, 0

    def _do_alloc(self, nbytes, user):
        self.calls += 1
        if self.at is not None and self.calls >= self.at:
            p = C.c_void_p()
            rc = self.lib.hipMalloc(C.byref(p), C.c_size_t(1 << 50))
            assert rc != 0 and not p.value
            self.refused += 1
            return None
        t = torch.empty(int(nbytes), dtype=torch.uint8, device="cuda")
        self.live[t.data_ptr()] = t
        return t.data_ptr()

    def _do_free(self, ptr, user):
        self.live.pop(ptr, None)


def test_refused_hipmalloc_does_not_fail_the_next_call(P):
    from paper_1606_02862_amd import _capi as A
    with P.Pic(workloads.reduced(3, 16, 16, 8), torch_alloc=False) as pic:
        one, z = np.ones(1), np.zeros(1, dtype=np.int32)
        d = one.ctypes.data_as(C.POINTER(C.c_double))
        rc = pic.lib.pic_rate_eval(pic.h, 0, 1, C.c_int64(1 << 45), d, d, z.ctypes.data_as(C.POINTER(C.c_int32)), d)
        assert rc == A.PIC_ERR_OOM
        pic.step(2)
        m = pic.moments()
        assert m["step"] == 2 and m["gauss_max"] <= 1e-4 * m["rho_max"]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("at", [1, 2, 3, 4])
def test_readback_without_scratch(P, at, precision):
    """The particles come back as with the scratch, and the next step runs."""
    cfg = workloads.config(2, nx=24, ny=16, nz=12, precision=precision)
    alloc = _Refusing(P)
    with P.Pic(cfg, allocator=alloc) as pic:
        pic.step(3)
        alloc.arm(None)
        want = [pic.get_particles(s) for s in range(2)]
        assert alloc.calls == 2 * 4
        held = len(alloc.live)
        alloc.arm(at)
        got = [pic.get_particles(s) for s in range(2)]
        assert alloc.refused >= 2 and len(alloc.live) == held
        alloc.arm(None)
        pic.step(1)
        assert pic.moments()["step"] == 4
    for a, b in zip(want, got):
        for k in a:
            assert np.array_equal(a[k], b[k]), k
