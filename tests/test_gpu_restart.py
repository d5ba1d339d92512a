"""Saved states of domains with pressure faces: the state as stored is what the next step starts
from, whatever densities the loading domain imposes, and saving, loading and timing the launch
configuration change nothing in it."""
import dataclasses

import numpy as np
import pytest

import oracle as O
from paper_2007_12266_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FIELDS = ("Na", "Nb", "phi", "rho", "ux", "uy", "uz")


@pytest.fixture(scope="module")
def lbm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2007_12266_amd import lbm as mod
    mod.load_library()
    return mod


def _prec(lbm, name):
    return {"fp64": lbm.FP64, "mixed": lbm.FP32_MIXED, "fp32dev": lbm.FP32_DEV}[name]


def _faces(inlet, rho_in=1.03, rho_out=0.97):
    """A displacement with an imposed inlet density, or an imposed inlet flux."""
    prob = inputs.displacement_problem(shape=(22, 18, 20), seed_geom=31, porosity_target=0.4,
                                       rho_in=rho_in, rho_out=rho_out)
    if inlet == "flux":
        n_in = int((prob.solid_mask()[0] == 0).sum())
        prob = dataclasses.replace(prob, inlet_mode=1, flux_in=0.01 * n_in)
    return prob


@pytest.mark.parametrize("mode", ["table", "rank", "compact"])
@pytest.mark.parametrize("inlet", ["density", "flux"])
@pytest.mark.parametrize("steps", [6, 7])
def test_state_loaded_under_other_face_densities_starts_as_stored(lbm, mode, inlet, steps):
    """A state stepped under one pair of densities (or under a flux inlet) is loaded into a domain
    that imposes others: its first step starts from the face populations in the state, and the new
    densities hold from the end of that step. FP64 against the oracle, which keeps the populations
    and changes its parameters, to 1e-12 of each field's largest value; alone and in a pool."""
    nm = {"table": lbm.NBR_TABLE, "rank": lbm.NBR_RANK, "compact": lbm.NBR_COMPACT}[mode]
    before, after = _faces(inlet), _faces("density", rho_in=1.01, rho_out=0.99)
    pore = before.solid_mask() == 0
    src = lbm.Domain(before, neighbour_mode=nm)
    blob = src.step(steps).save()
    solo = lbm.Domain(after, neighbour_mode=nm)
    pooled = lbm.Domain(after, neighbour_mode=nm)
    pool = lbm.Pool(1 << 32, precision=lbm.FP64, max_slots=1, chunk_steps=2)
    if steps % 2:
        pool.step(1)
    solo.load(blob)
    pooled.load(blob)
    assert solo.reduce() == src.reduce()
    pool.admit(pooled)
    ref = O.state_for(before).run(steps)
    ref.params = O.params_of(after)
    for n in (1, 1, 3):
        solo.step(n)
        pool.step(n)
        ref.run(n)
        gpu, want = solo.fields(), ref.fields()
        for k in FIELDS:
            scale = np.abs(want[k][pore]).max()
            assert np.abs(gpu[k][pore] - want[k][pore]).max() <= 1e-12 * scale, (k, n)
        assert pooled.save() == solo.save()
    pool.close()
    for d in (src, solo, pooled):
        d.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed", "fp32dev"])
@pytest.mark.parametrize("inlet", ["density", "flux"])
@pytest.mark.parametrize("steps", [0, 1, 2, 65, "morph"])
def test_saved_face_states_continue_and_save_again(lbm, inlet, precision, steps):
    """A state with pressure faces, initial, after an even or an odd step, or grown at its seventh,
    loads into another domain, saves as the same bytes, reads back the same fields and goes on bit
    for bit, also after the launch configuration was timed on it."""
    prob = _faces(inlet)
    a = lbm.Domain(prob, precision=_prec(lbm, precision))
    a.step(7 if steps == "morph" else steps)
    if steps == "morph":
        a.morph(delta=0.6)
    blob = a.save()
    b = lbm.Domain(prob, precision=_prec(lbm, precision))
    b.step(3)
    b.load(blob)
    assert b.save() == blob
    for name in ("Na", "phi", "rho", "uz"):
        assert np.array_equal(a.pore_field(name), b.pore_field(name))
    b.autotune(2)
    assert b.save() == blob
    for n in (1, 5, 64):
        assert a.step(n).save() == b.step(n).save()
    a.close()
    b.close()


@pytest.mark.parametrize("mode", ["table", "rank", "compact"])
@pytest.mark.parametrize("inlet", ["density", "flux"])
def test_single_plane_with_both_faces_matches_the_oracle(lbm, mode, inlet):
    """A domain of one plane, which is inlet and outlet at once (the inlet's condition first), alone
    and in a pool beside one whose faces the collide kernel applies: FP64 against the oracle, to
    1e-12 of each field's largest value (velocities: of the driven one's, about 0.04)."""
    rng = np.random.default_rng(12)
    shape = (1, 41, 34)
    prob = inputs.Problem(labels=(rng.random(shape) < 0.8).astype(np.int32),
                          label_kind=np.array([inputs.KIND_SOLID, inputs.KIND_PORE_INIT], np.int8),
                          label_affinity=np.array([0.3, 0.0]),
                          init_phi=inputs.bernoulli_phase(shape, 0.5, 13),
                          periodic=(True, True, False), force=(1e-4, 2e-4, 0.0), bc_z=1,
                          rho_in=1.01, rho_out=0.99)
    pore = prob.solid_mask() == 0
    if inlet == "flux":
        prob = dataclasses.replace(prob, inlet_mode=1, flux_in=1e-3 * int(pore.sum()))
    nm = {"table": lbm.NBR_TABLE, "rank": lbm.NBR_RANK, "compact": lbm.NBR_COMPACT}[mode]
    solo, pooled, mate = (lbm.Domain(p, neighbour_mode=nm) for p in (prob, prob, _faces("density")))
    pool = lbm.Pool(1 << 32, precision=lbm.FP64, max_slots=2, chunk_steps=4)
    pool.admit(pooled)
    pool.admit(mate)
    ref = O.state_for(prob)
    for n in (1, 6):
        ref.run(n)
        solo.step(n)
        pool.step(n)
        got, want = solo.fields(), ref.fields()
        for k in FIELDS:
            scale = np.abs(want["uz" if k[0] == "u" else k][pore]).max()
            # N_a is zero on a plane of the outlet's composition
            scale = max(scale, 1.0) if k[0] == "N" else scale
            assert np.abs(got[k][pore] - want[k][pore]).max() <= 1e-12 * scale, (k, n)
        assert pooled.save() == solo.save()
    pool.close()
    for d in (solo, pooled, mate):
        d.close()
