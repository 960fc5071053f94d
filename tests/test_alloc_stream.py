"""Device memory of a handle is asked for with the handle's stream current, in
pic_init and later (a readback's scratch), whatever stream the caller works on:
a stream-ordered allocator then hands out blocks that nothing queued on another
stream still uses."""
import contextlib
import ctypes as C
import types

import numpy as np
import pytest

import workloads

torch = pytest.importorskip("torch")


class _Recording:
    """Callbacks that note what `now()` is at every request."""

    def __init__(self, now, give):
        from paper_1606_02862_amd import _capi as A
        self.now, self.give, self.seen, self.freed = now, give, [], []
        self._alloc = A.ALLOC_FN(self._do_alloc)
        self._free = A.FREE_FN(self._do_free)
        self.struct = A.AllocT(self._alloc, self._free, None)

    def _do_alloc(self, nbytes, user):
        self.seen.append(self.now())
        return self.give(int(nbytes))

    def _do_free(self, ptr, user):
        self.freed.append(ptr)


def test_callbacks_run_with_the_handles_stream_current(monkeypatch):
    from paper_1606_02862_amd import pic as M
    caller, one, two = (types.SimpleNamespace(device="cuda:0", name=n) for n in ("caller", "one", "two"))
    current = [caller]

    @contextlib.contextmanager
    def stream(s):
        before, current[0] = current[0], s
        yield
        current[0] = before

    monkeypatch.setattr(torch.cuda, "stream", stream)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device: current[0])
    inner = _Recording(lambda: current[0].name, lambda n: 4096 if n == 256 else None)
    a, b = M._OnStream(inner, one), M._OnStream(inner, two)  # one allocator, two handles
    assert a.struct.alloc(256, None) == 4096 and b.struct.alloc(256, None) == 4096
    assert a.struct.alloc(512, None) is None
    assert inner.seen == ["one", "two", "one"] and current == [caller]
    current[0] = two
    assert b.struct.alloc(256, None) == 4096 and inner.seen[-1] == "two" and current == [two]
    a.struct.free(C.c_void_p(4096), None)
    assert inner.freed == [4096]


@pytest.mark.gpu
def test_scratch_of_a_handle_on_its_own_stream():
    import paper_1606_02862_amd as P
    P.load()
    live = {}

    def give(n):
        t = torch.empty(n, dtype=torch.uint8, device="cuda")
        live[t.data_ptr()] = t
        return t.data_ptr()

    alloc = _Recording(lambda: torch.cuda.current_stream().cuda_stream, give)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    cfg = workloads.reduced(3, 24, 16, 12)
    pics = [P.Pic(cfg, stream=s, allocator=alloc) for s in streams]
    for pic, s in zip(pics, streams):
        del alloc.seen[:]
        pic.step(2)
        p = pic.get_particles(0)
        n = len(p["id"])
        assert np.array_equal(p["id"], np.arange(n))
        pic.rate_eval("exact", 1, np.full(4, 50.0), np.full(4, 1e21), np.full(4, 2))
        assert len(alloc.seen) >= 6 and set(alloc.seen) == {s.cuda_stream}
        assert torch.cuda.current_stream().cuda_stream != s.cuda_stream
    for pic in pics:
        pic.close()
    assert set(alloc.freed) == set(live)
