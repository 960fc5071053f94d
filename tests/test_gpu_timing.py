"""pic_timing's launch count: launches of the particle kernel, of which species
without charge states share one on small grids, as those with them do."""
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("idx,box,per_cycle", [
    (2, (16, 16, 8), 1),    # electrons and protons together
    (3, (16, 16, 8), 2),    # electrons; ions with charge states
    (1, (16, 16, 8), 1),    # one species
    (2, (72, 64, 32), 2),   # 576 supercells: a launch for each species
])
def test_push_launches_counts_launches(idx, box, per_cycle):
    import paper_1606_02862_amd as P
    cfg = workloads.reduced(idx, *box)
    with P.Pic(cfg) as pic:
        n = sum(pic.count(s) for s in range(len(cfg["species"])))
        pic.timing(1)
        pic.step(3)
        pic.step(1)
        t = pic.timing(0)
    assert t["push_launches"] == 4 * per_cycle and t["push_particles"] == 4 * n
    assert t["push_ms"] > 0
