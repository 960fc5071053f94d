"""The particle kernel of one workgroup per supercell, which grids of more than
512 supercells run (here 576): arrivals of the previous cycle absorbed inside
the kernel for every shape, gather and precision and for ions with charge
states, the deterministic current of species of different scales, and the
overflow of the migration lists.  And steps in which one species runs it while
another runs several workgroups per supercell.

Tolerances: bit for bit where the deterministic option makes the cycle so;
1e-11 of the maximum in FP64 after a few cycles (FP64 atomics in any order);
elsewhere those of the one-step parity, 1e-5 of the momenta and 1e-4 of max |J|.
"""
import numpy as np
import pytest

import oracle
import workloads
from tests import parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BOX = dict(nx=72, ny=64, nz=32)


def _cfg(idx, shape, gather="standard", precision="fp32", **kw):
    cfg = workloads.config(idx, **BOX, shape=shape, gather=gather, precision=precision, **kw)
    for s in cfg["species"]:
        s.update(ppc=min(s["ppc"], 3), u_th=max(s["u_th"], 0.1))  # many leavers
        if precision == "fp64":
            s["ionize_into"] = -1
    return cfg


def _fields(seed):
    return workloads.random_fields(seed, BOX["nx"], BOX["ny"], BOX["nz"], amp=0.05)


def _run(cfg, calls):
    import paper_1606_02862_amd as P
    with P.Pic(cfg) as pic:
        if any(s["z_max"] for s in cfg["species"]):  # every charge state
            i = next(i for i, s in enumerate(cfg["species"]) if s["z_max"])
            p = pic.get_particles(i)
            p["zstate"] = (p["id"] % 7).astype(np.int32)
            pic.set_particles(i, p)
        E, B = _fields(17)
        pic.set_fields(E=E, B=B)
        for n in calls:
            pic.step(n)
        return pic.get_fields(), [pic.get_particles(s) for s in range(len(cfg["species"]))]


@pytest.mark.parametrize("idx,shape,gather,precision", [
    (1, "cic", "standard", "fp32"), (1, "cic", "galerkin", "fp32"), (2, "tsc", "standard", "fp32"),
    (2, "tsc", "galerkin", "fp32"), (1, "pcs", "standard", "fp32"), (1, "pcs", "galerkin", "fp32"),
    (3, "cic", "standard", "fp32"), (3, "tsc", "standard", "fp32"), (3, "pcs", "galerkin", "fp32"),
    (1, "cic", "standard", "fp64"), (2, "tsc", "galerkin", "fp64"), (3, "tsc", "standard", "fp64"), (1, "pcs", "standard", "fp64")])
def test_cycles_of_one_call_and_of_several(idx, shape, gather, precision):
    """A call of four cycles absorbs three cycles' arrivals in the particle
    kernel, four calls of one each cycle's in the migration kernel."""
    det = precision == "fp32"
    cfg = _cfg(idx, shape, gather, precision, **(dict(deterministic_j=True) if det else {}))
    (fa, pa), (fb, pb) = _run(cfg, [4]), _run(cfg, [1, 1, 1, 1])
    for a, b in zip(fa, fb):
        assert np.abs(a).max() > 0
        if det:
            assert np.array_equal(a, b)
        else:
            assert np.abs(a - b).max() <= 1e-11 * np.abs(b).max()
    for a, b in zip(pa, pb):
        assert np.array_equal(a["id"], b["id"]) and np.array_equal(a["zstate"], b["zstate"])
        for k, m in (("x", 72), ("y", 64), ("z", 32), ("ux", 0), ("uy", 0), ("uz", 0), ("w", 0)):
            if det:
                assert np.array_equal(a[k], b[k]), k
            else:
                d = np.abs(a[k] - b[k])
                assert np.minimum(d, np.abs(m - d)).max() <= 1e-11 * max(1.0, np.abs(b[k]).max()), k


@pytest.mark.parametrize("shape", ["cic", "tsc", "pcs"])
@pytest.mark.parametrize("det", [False, True])
def test_ions_and_unequal_scales_match_oracle(shape, det):
    """Electrons and carbon ions of every state, of different weight and charge:
    with the deterministic option the electrons' tiles are rescaled."""
    import paper_1606_02862_amd as P
    cfg = _cfg(3, shape, deterministic_j=det)
    cfg["species"][0]["ppc"], cfg["species"][1]["ppc"] = 2, 1
    st = oracle.init_state(cfg)
    st.E, st.B = _fields(18)
    st.species[1].zstate = (np.arange(len(st.species[1].x), dtype=np.int32) % 7).astype(np.int32)
    with P.Pic(cfg) as pic:
        s0 = parity.shared_start(pic, st)
        err = parity.one_step_errors(pic, cfg, s0)
    print(shape, det, err, flush=True)
    assert err["jmax"] > 0 and max(err["u"]) <= 1e-5 and max(err["x"]) <= 1e-5
    assert err["J"] <= 1e-4 and err["E"] <= 1e-4 and err["B"] <= 1e-4


@pytest.mark.parametrize("shape", ["cic", "tsc"])
def test_migration_overflow_is_reported(shape):
    """Every particle of one supercell leaves through one face in one step."""
    import paper_1606_02862_amd as P
    cfg = workloads.config(0, **BOX, shape=shape)
    with P.Pic(cfg) as pic:
        n = 2048
        r = workloads.rng(2)
        p = dict(x=r.uniform(7.9, 7.99, n), y=r.uniform(0, 8, n), z=r.uniform(0, 4, n), ux=np.full(n, 3.0),
                 uy=np.zeros(n), uz=np.zeros(n), w=np.full(n, 0.125), id=np.arange(n))
        pic.set_particles(0, p)
        with pytest.raises(P.PicError) as e:
            pic.step(2)
        assert e.value.code == -4
        q = pic.get_particles(0)  # what is left lies in the box
        for a, m in (("x", 72), ("y", 64), ("z", 32)):
            assert np.all(q[a] >= 0) and np.all(q[a] < m)
        pic.set_particles(0, dict(p, x=r.uniform(0, 72, n), ux=np.zeros(n)))
        pic.step(2)
        assert pic.count(0) == n


@pytest.mark.parametrize("shape", ["tsc", "pcs"])
@pytest.mark.parametrize("ppc", [(1, 8), (8, 1)])
def test_one_species_split_and_another_not(shape, ppc):
    """Few electrons beside many ions (of 12 supercells), and the reverse: TSC and
    PCS split the fuller species alone, each in a launch of its own."""
    import paper_1606_02862_amd as P
    cfg = workloads.config(3, nx=24, ny=16, nz=8, shape=shape)
    for s, n in zip(cfg["species"], ppc):
        s.update(ppc=n, u_th=0.1, coincident_with=-1)
    st = oracle.init_state(cfg)
    st.species[1].zstate = (np.arange(len(st.species[1].x), dtype=np.int32) % 7).astype(np.int32)
    st.E, st.B = workloads.random_fields(19, 24, 16, 8, amp=0.05)
    with P.Pic(cfg) as pic:
        s0 = parity.shared_start(pic, st)
        err = parity.one_step_errors(pic, cfg, s0)
        assert err["jmax"] > 0 and max(err["u"]) <= 1e-5 and max(err["x"]) <= 1e-5
        assert err["J"] <= 1e-4 and err["E"] <= 1e-4 and err["B"] <= 1e-4
        for n in (1, 5, 2):
            pic.step(n)
        for i, s in enumerate(st.species):
            assert np.array_equal(pic.get_particles(i)["id"], np.sort(s.id))
        assert pic.moments()["count"] == [len(s.id) for s in st.species]
    runs = []
    for det in (False, True):
        cfg["grid"]["deterministic_j"] = det
        with P.Pic(cfg) as pic:
            pic.step(3)
            runs.append(pic.get_fields())
    for a, b in zip(*runs):
        assert np.abs(a - b).max() <= 1e-4 * np.abs(b).max()
