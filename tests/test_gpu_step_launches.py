"""The fused sweep's launch carries the two-level steps and closes the step before; a call
of several steps, calls of one step and calls with every phase timed (each piece in a
launch of its own) give the same results bit for bit."""
import numpy as np
import pytest

from paper_2512_06173_amd import workloads as W

pytestmark = pytest.mark.gpu


def mlk():
    from paper_2512_06173_amd import mlk as m
    return m


def build(case, precision, tile):
    rng = np.random.default_rng(7)
    shape = (40, 33, 36)
    s = mlk().Simulation(shape, precision=precision, bc=("cpml",) * 6, cpml=(5,) * 6)
    s.set_eps(rng.choice([1.0, 2.25], size=(36, 33, 40)))
    if "tls" in case:
        n = {"tls": 1, "tls+": 700}[case["tls"]]
        t = W.tls_ensemble(rng, n, 9.0, 24.0, "superposition")
        s.add_tls(t.pos, t.sigma, t.gamma, t.omega0, t.dipole, t.rho0)
    if "ml" in case:
        m = W.random_multilevel(rng, 9, rng.uniform(9.0, 24.0, (9, 3)))
        s.add_multilevel(m.nlev, m.energies, m.mop, m.dipole, m.gphi, m.rho0, m.pos, m.sigma,
                         m.gamma)
    if "pole" in case:
        s.add_susceptibility((8, 8, 8, 20, 21, 22), 0.3, 0.01, 1.5)
    s.add_plane_source(2, 8, 1, 1.0, 0.3, 6.0, 2.0)
    s.add_probe(1, (20, 16, 18))
    s.add_probe(4, (12, 20, 9))
    if "flux" in case:
        s.add_flux_plane(*case["flux"])
    if "energy" in case:
        s.record_energy(3)
    s.record_populations(2)
    tx, ty, kz, lay = tile
    s.set_tile_width(tx)
    s.set_tuning(ty, kz)
    s.set_sweep_layers(lay if precision == "fp32" else 0)
    return s


CASES = [dict(tls="tls", flux=(2, 18)), dict(tls="tls+", ml=1, flux=(2, 31), energy=1),
         dict(ml=1, flux=(0, 20)), dict(tls="tls+", pole=1, flux=(1, 12)), dict(flux=(2, 9)),
         dict(tls="tls")]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("tile", [(64, 16, 8, 1), (32, 4, 3, 1), (64, 8, 16, 0), (32, 16, 64, 2)])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_one_call_equals_many_and_timed_ones(case, tile, precision):
    c, out = CASES[case], []
    for mode in range(3):
        s = build(c, precision, tile)
        if mode == 2:
            s.set_timing(True)
        for k in [9] if mode != 1 else [1, 3, 1, 4]:
            s.step(k)
        s.sync()
        r = s.fields() + [s.probe(0), s.probe(1), s.populations(), s.checkpoint_save()]
        if "flux" in c:
            r += [s.flux_series(), np.array(s.flux_total())]
        if "energy" in c:
            r.append(s.energy_series())
        out.append(r)
        s.close()
    assert np.any(out[0][1])  # the source has acted
    for o in out[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(out[0], o))


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_earliest_non_finite_step_is_reported(precision):
    """A probe beside an emitter sees a NaN at step 4 (through E) and the emitter's own state
    at step 5, in one launch: the earlier step is the one reported."""
    s = mlk().Simulation((24, 24, 24), precision=precision, bc=("periodic",) * 6)
    t = W.tls_ensemble(np.random.default_rng(2), 3, 10.0, 14.0, "superposition")
    s.add_tls(t.pos, t.sigma, t.gamma, t.omega0, t.dipole, t.rho0)
    s.add_probe(0, (2, 2, 2))
    s.step(4)
    s.sync()
    e = s.get_field(2)
    e[2, 4, 2] = np.nan  # reaches the probe in one step, the windows (7 to 17) later
    s.set_field(2, e)
    s.step(12)
    with pytest.raises(mlk().MlkError) as err:
        s.sync()
    first = int(str(err.value).split("step ")[1].split()[0].strip(".,"))
    p = s.probe(0)
    assert first == int(np.argmax(~np.isfinite(p))) and 4 <= first <= 6
    s.close()
