"""GPU-resident velocity Verlet vs the oracle's integrator; energy
conservation; skin/rebuild policy vs rebuilding every step."""
import numpy as np
import pytest
import torch

import oracle
import synthetic
import paper_2405_01491_amd as nnp
from paper_2405_01491_amd import md as nmd
from paper_2405_01491_amd import _lib
from tests.gpu_helpers import dev, to_dev

pytestmark = pytest.mark.gpu


def test_first_steps_track_oracle_trajectory(spec_bias):
    w = synthetic.workload(1)
    model = nnp.Model(spec_bias, "fp32")
    masses = synthetic.MASSES[w.species]
    v0 = nmd.maxwell_boltzmann(masses, 300.0, seed=5)
    pos, sp, _ = to_dev(w)
    sim = nmd.VelocityVerlet(model, pos.clone(), torch.from_numpy(v0).to(dev()), sp, masses, None, dt=0.5)
    for _ in range(10):
        sim.step()
    nl = oracle.neighbor_list(w.pos, None, None, 9.0)
    xr, vr, en = oracle.velocity_verlet(w.pos, v0, masses,
                                        lambda x: oracle.energy_forces_f64(x, w.species, None, spec_bias, nl),
                                        0.5, 10)
    x = sim.pos.cpu().numpy()
    v = sim.vel.cpu().numpy()
    print("10 steps: max |dx| %.3g A, max |dv| %.3g A/fs" % (np.abs(x - xr).max(), np.abs(v - vr).max()))
    assert np.abs(x - xr).max() < 1e-4
    assert np.abs(v - vr).max() < 1e-5
    assert abs(float(sim.e_mol[0]) - en[-1][0]) < 1e-4 * max(1.0, abs(en[-1][0]))


def test_nve_energy_conservation(spec):
    w = synthetic.geometry.small_water_box(64)
    model = nnp.Model(spec, "fp32")
    masses = synthetic.MASSES[w.species]
    pos, sp, _ = to_dev(w)
    v0 = torch.from_numpy(nmd.maxwell_boltzmann(masses, 300.0, seed=6)).to(dev())
    sim = nmd.VelocityVerlet(model, pos, v0, sp, masses, w.box, dt=0.25)
    E0 = sim.total_energy()
    Es = []
    for k in range(200):
        sim.step()
        if k % 20 == 19:
            Es.append(sim.total_energy())
    drift = max(abs(e - E0) for e in Es)
    ke = sim.kinetic_energy()
    print("NVE 200 steps: E0 %.6f drift %.3g eV (KE %.3g eV)" % (E0, drift, ke))
    assert drift < 0.02 * max(ke, 1.0)


def test_skin_policy_matches_rebuild_every_step(spec):
    w = synthetic.geometry.small_water_box(80)
    masses = synthetic.MASSES[w.species]
    v0 = nmd.maxwell_boltzmann(masses, 300.0, seed=7)
    res = []
    for skin, every in [(0.0, 1), (0.5, 20)]:
        model = nnp.Model(spec, "fp32")
        pos, sp, _ = to_dev(w)
        sim = nmd.VelocityVerlet(model, pos, torch.from_numpy(v0).to(dev()), sp, masses, w.box, dt=0.5,
                                 skin=skin, rebuild_every=every)
        for _ in range(40):
            sim.step()
        res.append((sim.pos.cpu().numpy(), float(sim.e_mol[0]), sim.rebuilds))
    # positions are wrapped at rebuilds: compare through the minimum image
    d = res[0][0] - res[1][0]
    d -= w.box * np.round(d / w.box)
    print("skin vs every-step after 40 steps: max |dx| %.3g A, rebuilds %d vs %d" % (np.abs(d).max(), res[0][2],
                                                                                    res[1][2]))
    assert np.abs(d).max() < 1e-4
    assert abs(res[0][1] - res[1][1]) < 1e-4 * max(1.0, abs(res[0][1]))
    assert res[1][2] < res[0][2]


def test_stage_profiling_counts(spec):
    w = synthetic.workload(1)
    model = nnp.Model(spec, "fp32")
    pos, sp, _ = to_dev(w)
    nmd.profile_enable(model, True)
    nl = nnp.nnp_neighbors(model, pos, None, 1, None, 5.1)
    for _ in range(3):
        nnp.nnp_energy_forces(model, pos, sp, None, 1, None, nl)
    st = nmd.profile_read(model)
    assert st["neighbors"][1] == 1 and st["aev"][1] == 3 and st["mlp"][1] == 3 and st["forces"][1] == 3
    assert all(v[0] >= 0 for v in st.values())


# ---------------------------------------------------------------- native engine (nnp_md_*)

def _engine(model, w, v0, **kw):
    pos, sp, _ = to_dev(w)
    return nmd.MDEngine(model, pos, torch.from_numpy(np.ascontiguousarray(v0)).to(dev()), sp,
                        synthetic.MASSES[w.species], w.box, **kw)


def _min_image(d, box):
    return d if box is None else d - box * np.round(d / box)


def test_engine_nve_tracks_oracle(spec_bias):
    w = synthetic.workload(1)
    model = nnp.Model(spec_bias, "fp32")
    masses = synthetic.MASSES[w.species]
    v0 = nmd.maxwell_boltzmann(masses, 300.0, seed=5)
    eng = _engine(model, w, v0, dt=0.5)
    eng.run(10)
    x, v, F, e = [t.cpu().numpy() for t in eng.state()]
    nl = oracle.neighbor_list(w.pos, None, None, 9.0)
    xr, vr, en = oracle.velocity_verlet(w.pos, v0, masses,
                                        lambda y: oracle.energy_forces_f64(y, w.species, None, spec_bias, nl),
                                        0.5, 10)
    print("engine NVE 10 steps: max |dx| %.3g A, max |dv| %.3g A/fs" % (np.abs(x - xr).max(), np.abs(v - vr).max()))
    assert np.abs(x - xr).max() < 1e-4 and np.abs(v - vr).max() < 1e-5
    assert abs(float(e[0]) - en[-1][0]) < 1e-4 * max(1.0, abs(en[-1][0]))
    assert eng.info()["steps"] == 10


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_engine_langevin_tracks_oracle(spec_bias, precision):
    w = synthetic.geometry.small_water_box(40)
    model = nnp.Model(spec_bias, precision)
    masses = synthetic.MASSES[w.species]
    v0 = nmd.maxwell_boltzmann(masses, 300.0, seed=8)
    eng = _engine(model, w, v0, dt=0.5, integrator="langevin", temperature=300.0, friction=20.0, seed=77,
                  skin=0.5, rebuild_every=5)
    eng.run(6)
    eng.run(4)                      # the noise stream continues across runs
    x, v, F, e = [t.cpu().numpy() for t in eng.state()]
    nl = oracle.neighbor_list(w.pos, None, w.box, 5.6)
    xr, vr, en = oracle.langevin_baoab(
        w.pos, v0, masses,
        lambda y: oracle.energy_forces_f64(y, w.species, w.box, spec_bias, nl,
                                           precision="bf16" if precision == "bf16" else "fp64"),
        0.5, 10, 300.0, 20.0, seed=77)
    dx = np.abs(_min_image(x - xr, w.box)).max()
    dv = np.abs(v - vr).max()
    print("engine Langevin %s 10 steps: max |dx| %.3g A, max |dv| %.3g A/fs, info %s"
          % (precision, dx, dv, eng.info()))
    tol = 1 if precision == "fp32" else 20
    assert dx < 1e-4 * tol and dv < 1e-5 * tol


@pytest.mark.parametrize("n_mol", [86, 190])
def test_engine_langevin_noise_of_several_blocks(spec_bias, n_mol):
    """Small systems' noise is drawn a step ahead, 256 atoms a block: 258 and
    570 atoms, against the oracle's noise; then a run cut at every step."""
    w = synthetic.geometry.small_water_box(n_mol)
    model = nnp.Model(spec_bias, "fp32")
    masses = synthetic.MASSES[w.species]
    v0 = nmd.maxwell_boltzmann(masses, 300.0, seed=8)
    kw = dict(dt=0.5, integrator="langevin", temperature=300.0, friction=20.0, seed=78, skin=0.5, rebuild_every=2)
    eng = _engine(model, w, v0, **kw)
    eng.run(3)
    x, v, _, _ = [t.cpu().numpy() for t in eng.state()]
    nl = oracle.neighbor_list(w.pos, None, w.box, 5.6)
    xr, vr, _ = oracle.langevin_baoab(
        w.pos, v0, masses, lambda y: oracle.energy_forces_f64(y, w.species, w.box, spec_bias, nl),
        0.5, 3, 300.0, 20.0, seed=78)
    assert np.abs(_min_image(x - xr, w.box)).max() < 1e-4 and np.abs(v - vr).max() < 1e-5
    cut = _engine(model, w, v0, **kw)
    for _ in range(3):
        cut.run(1)
    for a, b in zip(eng.state(), cut.state()):
        assert torch.equal(a, b)


def test_engine_split_runs_are_exact(spec):
    """A run cut into pieces gives bit-for-bit the state of one run of the
    same length: the noise is keyed by (step, atom), the rebuild decision and
    the list rows live on the device across calls."""
    w = synthetic.geometry.small_water_box(64)
    masses = synthetic.MASSES[w.species]
    v0 = nmd.maxwell_boltzmann(masses, 600.0, seed=9)
    out = []
    for pieces in ((30,), (10, 7, 13)):
        model = nnp.Model(spec, "fp32")
        eng = _engine(model, w, v0, dt=0.5, integrator="langevin", temperature=600.0, friction=5.0, seed=3,
                      skin=0.4, rebuild_every=5)
        for k in pieces:
            eng.run(k)
        out.append(([t.cpu() for t in eng.state()], eng.info()))
    print("info: one run %s, pieces %s" % (out[0][1], out[1][1]))
    assert out[0][1]["rebuilds"] == out[1][1]["rebuilds"] and out[0][1]["steps"] == 30
    for a, b in zip(out[0][0], out[1][0]):
        assert torch.equal(a, b)


def test_engine_nve_energy_log(spec):
    w = synthetic.geometry.small_water_box(64)
    model = nnp.Model(spec, "fp32")
    masses = synthetic.MASSES[w.species]
    v0 = nmd.maxwell_boltzmann(masses, 300.0, seed=6)
    eng = _engine(model, w, v0, dt=0.25, log_every=20, log_capacity=10)
    eng.run(200)
    rows = eng.log()
    assert rows.shape == (10, 2)
    tot = rows.sum(1)
    ke = rows[:, 1].mean()
    drift = np.abs(tot - tot[0]).max()
    print("engine NVE 200 steps: drift %.3g eV (KE %.3g eV)" % (drift, ke))
    assert drift < 0.02 * max(ke, 1.0)
    # the log's last row is the state's energies
    _, v, _, e = eng.state()
    assert abs(rows[-1, 0] - float(e[0])) < 1e-12 * max(1.0, abs(rows[-1, 0]))
    ke_now = float(0.5 * (torch.from_numpy(masses).double()[:, None] * v.cpu().double() ** 2).sum()
                   / nmd.ACC_UNIT)
    assert abs(rows[-1, 1] - ke_now) < 1e-6 * ke_now


def _zero_force_spec(spec):
    """The same model with every weight and bias zero: E is constant and every
    force is exactly zero, so the atoms are free particles."""
    import copy
    z = copy.copy(spec)
    z.weights = [[(np.zeros_like(W), np.zeros_like(b)) for W, b in layers] for layers in spec.weights]
    return z


@pytest.mark.parametrize("friction", [10.0, 100.0])
def test_engine_langevin_equipartition(spec, friction):
    """Free particles under BAOAB (zero forces) relax from rest to the bath:
    <KE> = 3N/2 kT.  For free particles the O step is an exact
    Ornstein-Uhlenbeck update, so the mean is exact at any step size and
    the gate is set by sampling error alone: N = 3,000 atoms, samples one
    or more velocity-correlation times (1 / (2 gamma)) apart after a burn-in
    of 5 / gamma."""
    w = synthetic.geometry.small_water_box(1000)
    model = nnp.Model(_zero_force_spec(spec), "fp32")
    v0 = np.zeros((w.n_atoms, 3), np.float32)
    every = max(1, int(round(1e3 / (2.0 * friction) / 0.5)))       # 1 / (2 gamma) in 0.5 fs steps
    burn = int(round(5e3 / friction / 0.5))
    n_samples = 40
    eng = _engine(model, w, v0, dt=0.5, integrator="langevin", temperature=300.0, friction=friction, seed=31,
                  skin=0.5, rebuild_every=20, log_every=every, log_capacity=(burn // every) + n_samples + 2)
    eng.run(burn + every * n_samples)
    rows = eng.log()
    assert np.all(rows[:, 0] == 0.0)                                # constant energy: the zero model
    ke = rows[-n_samples:, 1]
    want = 1.5 * w.n_atoms * nmd.KB_EV * 300.0
    # one sample's relative standard deviation is sqrt(2 / 3N) = 1.5 %; the mean of 40 is near 0.3 %
    sem = np.std(ke, ddof=1) / np.sqrt(n_samples) / want
    print("Langevin %.0f/ps free particles: <KE> %.5f eV, 3N kT/2 %.5f eV (ratio %.4f, sem %.4f)"
          % (friction, ke.mean(), want, ke.mean() / want, sem))
    assert abs(ke.mean() / want - 1.0) < 0.015
    _, v, F, _ = eng.state()
    assert float(F.abs().max()) == 0.0


@pytest.mark.parametrize("n_mol", [64, 3000])
def test_engine_forces_equal_plain_path(spec_bias, n_mol):
    """The engine's last kernel gathers each atom's force with the same
    per-row sum as the plain path's gather, so at the same positions and
    list the forces agree bit for bit (both the fused small-system step and
    the general step above 8,192 atoms); the float64 potential energy, summed
    in another fixed order, agrees to rounding."""
    w = synthetic.geometry.small_water_box(n_mol)
    model = nnp.Model(spec_bias, "fp32")
    masses = synthetic.MASSES[w.species]
    v0 = nmd.maxwell_boltzmann(masses, 300.0, seed=14)
    eng = _engine(model, w, v0, dt=0.5)                 # no skin: rebuilt (and wrapped) every step
    eng.run(3)
    x, _, F, e = eng.state()
    sp = torch.from_numpy(w.species).to(dev())
    nl = nnp.nnp_neighbors(model, x, None, 1, w.box, model.spec.rc_r)
    e2, _, F2 = nnp.nnp_energy_forces(model, x, sp, None, 1, w.box, nl)
    print("engine vs plain path, %d atoms: max |dF| %.3g, dE %.3g eV"
          % (w.n_atoms, float((F - F2).abs().max()), float(e[0] - e2[0])))
    assert torch.equal(F, F2)
    assert abs(float(e[0]) - float(e2[0])) <= 1e-12 * max(1.0, abs(float(e2[0])))


def test_engine_general_path_tracks_oracle(spec_bias):
    """Above 8,192 atoms the engine runs the general multi-kernel step (its own
    integrator kernel; the rebuild decision and the wrap inside the binning
    kernel of the periodic box)."""
    w = synthetic.geometry.water_box(3000, seed=21)          # 9,000 atoms
    model = nnp.Model(spec_bias, "fp32")
    masses = synthetic.MASSES[w.species]
    v0 = nmd.maxwell_boltzmann(masses, 300.0, seed=22)
    eng = _engine(model, w, v0, dt=0.5, integrator="langevin", temperature=300.0, friction=10.0, seed=5,
                  skin=0.5, rebuild_every=3)
    eng.run(4)
    x, v, F, e = [t.cpu().numpy() for t in eng.state()]
    nl = oracle.neighbor_list(w.pos, None, w.box, 5.6)
    xr, vr, en = oracle.langevin_baoab(
        w.pos, v0, masses, lambda y: oracle.energy_forces_f64(y, w.species, w.box, spec_bias, nl),
        0.5, 4, 300.0, 10.0, seed=5)
    dx = np.abs(_min_image(x - xr, w.box)).max()
    dv = np.abs(v - vr).max()
    print("engine general path 4 steps: max |dx| %.3g A, max |dv| %.3g A/fs, |dE| %.3g eV, info %s"
          % (dx, dv, abs(float(e[0]) - en[-1][0]), eng.info()))
    assert dx < 1e-4 and dv < 1e-5
    assert abs(float(e[0]) - en[-1][0]) < 1e-5 * max(1.0, abs(en[-1][0]))


def test_engine_open_general_path_tracks_oracle(spec_bias):
    """An open system above 8,192 atoms: the rebuild decision and the new
    reference run as kernels of their own (the binning kernel takes them only
    for periodic boxes).  Rebuilt every second step."""
    wb = synthetic.geometry.water_box(3000, seed=23)          # 9,000 atoms, taken without the box
    w = synthetic.geometry.Workload("water_cube_open_9000", wb.pos, wb.species, wb.mol, wb.n_mol, None)
    model = nnp.Model(spec_bias, "fp32")
    masses = synthetic.MASSES[w.species]
    v0 = nmd.maxwell_boltzmann(masses, 300.0, seed=24)
    eng = _engine(model, w, v0, dt=0.5, skin=0.5, rebuild_every=2)
    eng.run(4)
    x, v, F, e = [t.cpu().numpy() for t in eng.state()]
    nl = oracle.neighbor_list(w.pos, None, None, 5.6)
    xr, vr, en = oracle.velocity_verlet(w.pos, v0, masses,
                                        lambda y: oracle.energy_forces_f64(y, w.species, None, spec_bias, nl),
                                        0.5, 4)
    info = eng.info()
    print("engine open general path 4 steps: max |dx| %.3g A, max |dv| %.3g A/fs, |dE| %.3g eV, info %s"
          % (np.abs(x - xr).max(), np.abs(v - vr).max(), abs(float(e[0]) - en[-1][0]), info))
    assert np.abs(x - xr).max() < 1e-4 and np.abs(v - vr).max() < 1e-5
    assert abs(float(e[0]) - en[-1][0]) < 1e-5 * max(1.0, abs(en[-1][0]))
    assert info["steps"] == 4 and info["rebuilds"] >= 3


@pytest.mark.parametrize("n_mol", [64, 3000])
def test_engine_nonfinite_velocity_is_flagged(spec, n_mol):
    """A non-finite velocity makes the step's displacement infinite, so the
    list is rebuilt and the rebuild flags the coordinate: the run returns
    NNP_E_NONFINITE, and the steps it enqueued still count (the engine's state
    slots and noise counters follow them).  192 atoms take the fused front
    kernel, 9,000 the binning kernel's decision."""
    w = synthetic.geometry.water_box(n_mol, seed=41)
    model = nnp.Model(spec, "fp32")
    masses = synthetic.MASSES[w.species]
    v0 = nmd.maxwell_boltzmann(masses, 300.0, seed=42)
    v0[7, 1] = np.nan
    eng = _engine(model, w, v0, dt=0.5, skin=0.5, rebuild_every=20)
    with pytest.raises(nnp.NNPError) as e:
        eng.run(3)
    assert e.value.status == _lib.NNP_E_NONFINITE
    assert eng.info()["steps"] == 3


@pytest.mark.parametrize("case", ["faces_periodic_3cells", "boundary_cutoff_3cells"])
def test_engine_forces_equal_plain_path_adversarial(spec_bias, case):
    """The builder's adversarial boxes at the engine's list radius (atoms on
    the faces, at L - ulp and outside the box; pairs across the periodic
    boundary within two ulp of r_list): the engine's set-up (wrap into the
    box, fixed-stride rows, reverse index from the AEV kernel, force gather)
    and one step (the fused front's wrap and binning, the row kernel, the
    last kernel's gather) give the plain path's forces bit for bit at the
    engine's own positions."""
    model = nnp.Model(spec_bias, "fp32")
    w = next(c for c in synthetic.geometry.adversarial_cases(r_list=float(model.spec.rc_r)) if c.name == case)
    v0 = np.zeros((w.n_atoms, 3), np.float32)
    eng = _engine(model, w, v0, dt=0.01)                # no skin: the list is rebuilt every step
    sp = torch.from_numpy(w.species).to(dev())
    for k in range(2):
        x, _, F, _ = eng.state()
        assert bool(((x >= 0) & (x < torch.from_numpy(w.box).to(dev()))).all())   # wrapped into the box
        nl = nnp.nnp_neighbors(model, x, None, 1, w.box, model.spec.rc_r)
        _, _, F2 = nnp.nnp_energy_forces(model, x, sp, None, 1, w.box, nl)
        print("%s, after %d steps: %d pairs, max |F| %.3g, max |dF| %.3g"
              % (case, k, nl.n_pairs, float(F2.abs().max()), float((F - F2).abs().max())))
        assert torch.isfinite(F).all()
        assert torch.equal(F, F2)
        eng.run(1)
