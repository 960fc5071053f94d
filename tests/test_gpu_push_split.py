"""The particle kernel with several workgroups per supercell (grids of at most
512 supercells) and with one: one step against the FP64 oracle on either side
of the rule, for every shape, precision and gather, with ions (charge states)
among the species, and particle numbers that leave a last frame partial.  A
crowded box makes many parts with uneven shares and thousands of leavers.

Tolerances are those of the one-step parity elsewhere: 1e-5 of the momenta and
1e-4 of max |J| in FP32, 1e-12 in FP64.
"""
import numpy as np
import pytest

import oracle
import workloads
from tests import parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BOXES = [(8, 8, 4), (24, 16, 12), (64, 64, 32), (72, 64, 32)]  # 1, 18, 512 and 576 supercells


def _check(cfg, err, jtol=1e-4):
    fp64 = cfg["grid"].get("precision") == "fp64"
    print(cfg["grid"]["shape"], err, flush=True)
    assert err["jmax"] > 0
    assert max(err["u"]) <= (1e-12 if fp64 else 1e-5) and max(err["x"]) <= (1e-12 if fp64 else 1e-5)
    tol = 1e-12 if fp64 else jtol
    assert err["J"] <= tol and err["E"] <= tol and err["B"] <= tol


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shape,gather", [("cic", "standard"), ("tsc", "standard"), ("pcs", "standard"), ("tsc", "galerkin")])
@pytest.mark.parametrize("box", BOXES)
def test_one_step_on_either_side_of_the_rule(box, shape, gather, precision):
    import paper_1606_02862_amd as P
    cfg = workloads.config(2, nx=box[0], ny=box[1], nz=box[2], shape=shape, gather=gather, precision=precision)
    for s in cfg["species"]:
        s["ppc"] = 3
        s["u_th"] = 0.1  # many crossers and leavers
    st = oracle.init_state(cfg)
    with P.Pic(cfg) as pic:
        g = np.random.default_rng(9)
        st.E, st.B = (0.05 * g.standard_normal(st.E.shape) for _ in range(2))
        s0 = parity.shared_start(pic, st)
        _check(cfg, parity.one_step_errors(pic, cfg, s0))


@pytest.mark.parametrize("shape", ["cic", "tsc"])
def test_ions_with_charge_states(shape):
    import paper_1606_02862_amd as P
    cfg = workloads.config(3, nx=16, ny=16, nz=8, shape=shape)
    st = oracle.init_state(cfg)
    oracle.step(st, 3)
    st.species[1].zstate = (np.arange(len(st.species[1].x), dtype=np.int32) % 7).astype(np.int32)
    with P.Pic(cfg) as pic:
        s0 = parity.shared_start(pic, st)
        _check(cfg, parity.one_step_errors(pic, cfg, s0))


@pytest.mark.parametrize("shape", ["cic", "tsc", "pcs"])
def test_uneven_supercells(shape):
    """Most particles in one supercell of four, fast: its parts run several
    frames each while the others' have nothing to do."""
    import paper_1606_02862_amd as P
    cfg = workloads.config(1, nx=16, ny=16, nz=4, shape=shape)
    cfg["species"][0]["cap_ppc"] = 64
    st = oracle.init_state(cfg)
    s = st.species[0]
    g = np.random.default_rng(4)
    n = len(s.x)
    crowd = g.random(n) < 0.3
    s.x[crowd], s.y[crowd] = 8 * g.random(crowd.sum()), 8 * g.random(crowd.sum())
    for a in ("ux", "uy", "uz"):
        setattr(s, a, 0.5 * g.standard_normal(n))
    with P.Pic(cfg) as pic:
        s0 = parity.shared_start(pic, st)
        err = parity.one_step_errors(pic, cfg, s0)
        _check(cfg, err)
        pic.step(3)
        assert pic.count(0) == n
        assert np.array_equal(pic.get_particles(0)["id"], np.arange(n))


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", ["cic", "tsc", "pcs"])
def test_species_that_share_a_launch(shape, precision):
    """Three species without charge states of different density and mass in one
    launch, and (FP32) one with, in another; an immobile one in neither."""
    import paper_1606_02862_amd as P
    cfg = workloads.config(3, nx=24, ny=16, nz=8, shape=shape, precision=precision)
    el, ion = cfg["species"]
    plain = dict(el, coincident_with=-1, cap_ppc=None)
    species = [dict(plain, ppc=5, u_th=0.1), dict(plain, name="light", charge=0.5, mass=3.0, ppc=2, density=0.3, u_th=0.05),
               dict(plain, name="proton", charge=1.0, mass=1836.0, ppc=7, density=0.9, u_th=0.002)]
    species.append(dict(plain, name="fixed", charge=1.0, ppc=2, mobile=False) if precision == "fp64" else dict(ion, ionize_into=0))
    cfg["species"] = species
    st = oracle.init_state(cfg)
    g = np.random.default_rng(8)
    st.E, st.B = (0.05 * g.standard_normal(st.E.shape) for _ in range(2))
    with P.Pic(cfg) as pic:
        s0 = parity.shared_start(pic, st)
        _check(cfg, parity.one_step_errors(pic, cfg, s0))


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("box", [(16, 16, 8), (72, 64, 32)])
def test_large_ids_survive_migration(box, precision):
    """Ids whose bits read as NaN, infinity and negative floats travel through the
    arrival records (as the fourth real of one) unchanged."""
    import paper_1606_02862_amd as P
    cfg = workloads.config(1, nx=box[0], ny=box[1], nz=box[2], shape="cic", precision=precision)
    cfg["species"][0].update(ppc=2, u_th=0.5)
    with P.Pic(cfg) as pic:
        p = pic.get_particles(0)
        n = len(p["id"])
        base = np.array([0x7F800000, 0x7FC00000, 0xFF800000, 0xFFFFFFFF - n], dtype=np.int64)
        p["id"] = base[np.arange(n) % 4] + np.arange(n) // 4
        pic.set_particles(0, p)
        for k in (1, 3, 4):
            pic.step(k)
        q = pic.get_particles(0)
    order = np.argsort(p["id"])
    assert np.array_equal(q["id"], p["id"][order])
    assert np.array_equal(q["w"], p["w"][order])
    moved = np.floor(q["x"] / 8) != np.floor(p["x"][order] / 8)
    assert moved.sum() > n // 10
