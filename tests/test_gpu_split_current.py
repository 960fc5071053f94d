"""The current of a supercell that several workgroups deposit (grids of few
supercells): one exact fixed-point sum, rounded to FP32 once, as with one
workgroup.  The weights here make the fixed-point scale a power of two, so
PIC_OPT_DETERMINISTIC_J, whose J is that exact sum over all supercells rounded
once, must be met bit for bit, cycle after cycle.  Partial tiles rounded one by
one and added in FP32, in any order, miss it in the last place of many nodes.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _run(cfg, det, cycles):
    import paper_1606_02862_amd as P
    cfg["grid"]["deterministic_j"] = det
    with P.Pic(cfg) as pic:
        out = []
        for n in cycles:
            pic.step(n)
            out.append(pic.get_fields())
        parts = [pic.get_particles(s) for s in range(len(cfg["species"]))]
    return out, parts


@pytest.mark.parametrize("shape", ["cic", "tsc", "pcs"])
@pytest.mark.parametrize("box", [(8, 8, 4), (16, 16, 16)])
def test_parts_of_a_supercell_add_up_exactly(box, shape):
    cfg = workloads.config(0, nx=box[0], ny=box[1], nz=box[2], shape=shape)
    cfg["species"][0].update(ppc=16, u_th=0.1)
    a, pa = _run(cfg, False, (1, 1, 3))
    b, pb = _run(cfg, True, (1, 1, 3))
    for (E, B, J), (E1, B1, J1) in zip(a, b):
        assert np.abs(J).max() > 0
        assert np.array_equal(J, J1) and np.array_equal(E, E1) and np.array_equal(B, B1)
    for k in pa[0]:
        assert np.array_equal(pa[0][k], pb[0][k]), k


def test_species_of_several_parts_and_of_one():
    """Electrons of several parts beside ions of one that share their launch:
    the ions' tiles, rounded once per supercell, and the electrons' exact sums
    reach one J, and none is left over for the next cycle."""
    cfg = workloads.config(2, nx=32, ny=32, nz=16)
    cfg["species"][0].update(ppc=32, u_th=0.1)
    cfg["species"][1].update(ppc=1, u_th=0.001)
    a, _ = _run(cfg, False, (1, 2, 1))
    b, _ = _run(cfg, True, (1, 2, 1))
    # roundings of one cycle: per species and tile (at most 8 tiles a node), 2^-24 of J
    # each; later cycles compound FP32 rounding of positions and fields
    for k, ((E, B, J), (E1, B1, J1)) in enumerate(zip(a, b)):
        assert np.abs(J - J1).max() <= (32 * 2.0**-24 if k == 0 else 1e-4) * np.abs(J1).max()
