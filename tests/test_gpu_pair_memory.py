"""Memory of the ionisation step's (cell, charge state) pairs: no more of them
than ion slots, whatever the number of states, and full slabs in which every ion
is a pair of its own rated right (the last pair of a supercell included)."""
import numpy as np
import pytest

import oracle
import workloads
from oracle import ionize
from tests import parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _cfg(box, z_max, ppc, cap):
    cfg = workloads.reduced(3, *box)
    cfg["grid"]["shape"] = "cic"
    ion = cfg["species"][1]
    ion.update(ppc=ppc, cap_ppc=cap, z_init=0, z_max=z_max, ionize_into=0,
               ionization_ev=tuple(10.0 * (z + 1) for z in range(z_max)), lotz_q=(1,) * z_max)
    return cfg


def test_bytes_of_a_handle_with_many_states_and_few_ions():
    import paper_1606_02862_amd as P
    asked = []

    class Noting(P.pic.TorchAllocator):
        def _do_alloc(self, nbytes, user):
            asked.append(nbytes)
            return super()._do_alloc(nbytes, user)

    box = (32, 32, 16)
    with P.Pic(_cfg(box, 7, 1, 1), allocator=Noting(torch.device("cuda:0"))):
        many = sum(asked)
    del asked[:]
    with P.Pic(_cfg(box, 1, 1, 1), allocator=Noting(torch.device("cuda:0"))):
        one = sum(asked)
    # one ion slot per cell: both have a pair a slot
    print("bytes", many, one, flush=True)
    assert many == one


@pytest.mark.parametrize("mode,staged", [("exact", False), ("exact", True), ("table", False)])
def test_every_slot_a_pair(mode, staged):
    """Slabs filled to the last slot, ions of one cell in different states."""
    import paper_1606_02862_amd as P
    box, cap = (16, 8, 8), 2
    cfg = _cfg(box, 7, cap, cap)
    cfg["grid"]["n_ref_cm3"] = 1e25
    n_c = box[0] * box[1] * box[2] * cap
    n_e = box[0] * box[1] * box[2] * cfg["species"][0]["ppc"]
    st = oracle.init_state(cfg)
    s = st.species[1]
    cell = np.floor(s.x).astype(int) + 16 * (np.floor(s.y).astype(int) + 8 * np.floor(s.z).astype(int))
    nth = np.zeros(n_c, dtype=int)
    for c in range(box[0] * box[1] * box[2]):
        k = np.nonzero(cell == c)[0]
        nth[k] = np.arange(len(k))
    s.zstate = ((cell + 3 * nth) % 7).astype(np.int32)
    assert len(set(zip(cell, s.zstate))) == n_c
    with P.Pic(cfg) as pic:
        s0 = parity.shared_start(pic, st)
        s0.step = 0
        ref = s0.copy()
        d = ionize.ionize_step(ref, cfg, 0, 1, n_e + n_c, n_e, return_details=True)
        stats = pic.ionize(mode, staged=staged)
        got = parity.pull_state(pic, s0)
    assert stats["ions_active"] == n_c and d["fire"].sum() > n_c // 20
    tol = 1e-12 if mode == "exact" else 3e-8
    for k in np.nonzero(got.species[1].zstate != ref.species[1].zstate)[0]:
        assert abs(d["uniforms"][k] - d["prob"][k]) < tol * max(d["prob"][k], 1e-300)
