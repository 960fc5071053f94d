"""Ionisation from cells that hold ions of several charge states: the step rates
each (cell, state) pair once, so every ion must still get the rate of its own
cell and state.  All ions of a reduced carbon box take states 0..6 in turn (6 is
past the last ionising state) and are compared with the FP64 oracle: the same
decisions on the same uniforms, for one supercell and for several, through the
fused and the staged step.
"""
import numpy as np
import pytest

import oracle
import workloads
from oracle import ionize
from tests import parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("box", [(8, 8, 4), (24, 16, 8)])
@pytest.mark.parametrize("mode,staged", [("exact", False), ("exact", True), ("table", False)])
def test_mixed_states_match_oracle(box, mode, staged):
    import paper_1606_02862_amd as P
    cfg = workloads.reduced(3, *box)
    cfg["grid"]["n_ref_cm3"] = 1e26  # nu dt ~ 1 for the low states
    n_e0, n_c0 = (box[0] * box[1] * box[2] * cfg["species"][s]["ppc"] for s in (0, 1))
    st = oracle.init_state(cfg)
    oracle.step(st, 4)
    st.species[1].zstate = (np.arange(n_c0, dtype=np.int32) * 5 % 7).astype(np.int32)
    with P.Pic(cfg) as pic:
        s0 = parity.shared_start(pic, st)
        s0.step = 0
        ref = s0.copy()
        d = ionize.ionize_step(ref, cfg, 0, 1, n_e0 + n_c0, n_e0, return_details=True)
        stats = pic.ionize(mode, staged=staged)
        got = parity.pull_state(pic, s0)
    fire = d["fire"]
    assert stats["ions_active"] == int((s0.species[1].zstate < 6).sum())
    assert fire.sum() > 100 * box[0] * box[1] * box[2] / 1024
    # the table's rate is within 3e-8 of the quadrature's
    tol = 1e-12 if mode == "exact" else 3e-8
    differ = np.nonzero(got.species[1].zstate != ref.species[1].zstate)[0]
    for k in differ:
        assert abs(d["uniforms"][k] - d["prob"][k]) < tol * max(d["prob"][k], 1e-300)
    if len(differ) == 0:
        assert stats["ionized"] == int(fire.sum())
        ref.species[0].sort_by_id()
        assert np.array_equal(got.species[0].id, ref.species[0].id)
