"""Readback of few particles: sorted by the host, with no device scratch asked
for; from more than 8192 slots on ranked by the GPU.  The order and the values
are the same on either side."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("cap,scratch", [(8, False), (10, True)])  # 8 ppc: 4 supercells of 2048 slots, and of 2560
def test_route_and_order(cap, scratch, precision):
    import paper_1606_02862_amd as P

    class Counting(P.pic.TorchAllocator):
        calls = 0

        def _do_alloc(self, nbytes, user):
            Counting.calls += 1
            return super()._do_alloc(nbytes, user)

    cfg = workloads.config(2, nx=16, ny=16, nz=4, precision=precision)
    for s in cfg["species"]:
        s.update(ppc=3, cap_ppc=cap)
    g = np.random.default_rng(5)
    with P.Pic(cfg, allocator=Counting(torch.device("cuda:0"))) as pic:
        n = pic.count(1)
        p = pic.get_particles(1)
        p["id"] = g.permutation(5 * n)[:n].astype(np.int64)
        pic.set_particles(1, p)
        before = Counting.calls
        q = pic.get_particles(1)
        assert (Counting.calls > before) == scratch
    order = np.argsort(p["id"])
    for k in p:
        assert np.array_equal(p[k][order], q[k]), k
