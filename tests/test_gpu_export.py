"""get_particles in id order: ids ranked on the GPU (dense, with gaps, at the
ends of 32-id words and of the rank kernel's blocks), and the cases that sort
on the host (duplicate ids, ids far apart), for FP32 and FP64 handles.  Every
value must come back with its id, exactly."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _ids(kind, n, g):
    if kind == "dense":
        return g.permutation(n)
    if kind == "gaps":  # every 3rd id, and the last of a 1024-word block
        return np.concatenate([g.permutation(n - 2) * 3, [32 * 1024 * 9 - 1, 32 * 1024 * 9]])
    if kind == "sparse":
        return np.concatenate([g.permutation(n - 1), [2**32 - 1]])
    return np.concatenate([g.permutation(n - 5), np.full(5, 7)])  # duplicates


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("kind", ["dense", "gaps", "sparse", "duplicates"])
@pytest.mark.parametrize("n", [33, 60_000])
def test_particles_come_back_in_id_order(n, kind, precision):
    import paper_1606_02862_amd as P
    cfg = workloads.reduced(3, 24, 16, 12)
    if precision == "fp64":
        cfg["grid"]["precision"] = "fp64"
        cfg["species"][1]["ionize_into"] = -1
    cfg["species"][1]["cap_ppc"] = 64
    g = np.random.default_rng(6)
    rt = np.float64 if precision == "fp64" else np.float32
    box = dict(x=24, y=16, z=12)
    p = {k: (g.random(n, dtype=np.float32) * 0.999 * m).astype(np.float32).astype(np.float64) for k, m in box.items()}
    p.update({k: g.standard_normal(n).astype(rt) for k in ("ux", "uy", "uz", "w")})
    p["id"] = _ids(kind, n, g).astype(np.int64)
    p["zstate"] = g.integers(0, 7, n).astype(np.int32)
    with P.Pic(cfg) as pic:
        pic.set_particles(1, p)
        got = pic.get_particles(1)
    assert np.array_equal(got["id"], np.sort(p["id"]))
    # by id, and by position among equal ids
    a = np.lexsort((p["x"], p["id"]))
    b = np.lexsort((got["x"], got["id"]))
    for k in ("ux", "uy", "uz", "w", "zstate"):
        assert np.array_equal(p[k][a], got[k][b]), k
    for k in box:  # positions are held relative to the supercell, in the handle's precision
        assert np.abs(p[k][a] - got[k][b]).max() <= (0 if precision == "fp64" else 2.0 ** -21)
