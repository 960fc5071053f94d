"""The field update of one cycle against the same Yee update in FP64 torch, from
the cycle's own J: on a box of one supercell (every neighbour wraps onto it),
ragged boxes, and one on either side of the size at which the update changes
from two fused kernels to three passes in place.

Tolerance: each new value is a handful of FP32 (FP64) operations on numbers no
larger than the largest field or dt J, so 16 roundings of that size bound it.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _curl(F, forward):
    def diff(a, axis):
        return torch.roll(a, -1, 2 - axis) - a if forward else a - torch.roll(a, 1, 2 - axis)
    return torch.stack([diff(F[2], 1) - diff(F[1], 2), diff(F[0], 2) - diff(F[2], 0), diff(F[1], 0) - diff(F[0], 1)])


def _config(box, precision, det=False):
    cfg = workloads.reduced(0, *box)
    cfg["grid"]["precision"] = precision
    cfg["grid"]["deterministic_j"] = det
    cfg["species"][0]["ppc"] = 2
    return cfg


def _start(pic, box, precision):
    g = np.random.default_rng(3)
    rt = np.float64 if precision == "fp64" else np.float32
    E, B = ((0.02 * g.standard_normal((3, box[2], box[1], box[0]))).astype(rt) for _ in range(2))
    pic.set_fields(E=E, B=B, J=np.ones_like(E))
    return E, B


# the last two of each: either side of 3 MiB per field component
@pytest.mark.parametrize("box,precision", [(b, p) for p, ends in (("fp32", [(128, 96, 64), (136, 96, 64)]),
                                                                  ("fp64", [(96, 64, 64), (104, 64, 64)]))
                                           for b in [(8, 8, 4), (40, 24, 12), *ends]])
def test_update_matches_torch(box, precision):
    import paper_1606_02862_amd as P
    cfg = _config(box, precision)
    dt = cfg["grid"]["dt"]
    with P.Pic(cfg) as pic:
        E, B = _start(pic, box, precision)
        for _ in range(2):
            pic.step(1)
            E1, B1, J1 = pic.get_fields()
            e, b, j = (torch.from_numpy(a).double() for a in (E, B, J1))
            assert np.abs(J1).max() < 1.0 and np.abs(J1).max() > 0.0
            b = b - 0.5 * dt * _curl(e, True)
            e = e + dt * (_curl(b, False) - j)
            b = b - 0.5 * dt * _curl(e, True)
            tol = 16 * (2.0 ** -53 if precision == "fp64" else 2.0 ** -24) * max(np.abs(E).max(), np.abs(B).max(), np.abs(J1).max())
            assert float((e - torch.from_numpy(E1)).abs().max()) < tol
            assert float((b - torch.from_numpy(B1)).abs().max()) < tol
            E, B = E1, B1


@pytest.mark.parametrize("box", [(24, 16, 8), (136, 128, 64)])
def test_calls_of_one_and_of_several_cycles_agree(box):
    """Order-independent sums: three calls of one cycle, with and without the
    timing that separates the migration, equal one call of three bit for bit."""
    import paper_1606_02862_amd as P
    cfg = _config(box, "fp32", det=True)
    out = []
    for calls, timed in (((3,), False), ((1, 1, 1), False), ((2, 1), True)):
        with P.Pic(cfg) as pic:
            _start(pic, box, "fp32")
            if timed:
                pic.timing(1)
            for n in calls:
                pic.step(n)
            p = pic.get_particles(0)
            out.append([*pic.get_fields(), p["id"], p["x"], p["uz"]])
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert np.array_equal(a, b)
