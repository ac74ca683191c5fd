"""Emitter launches at their edges: mixed and single level counts around a wavefront's 64
emitters, Hamiltonians with degenerate and with tiny levels, and classical-path calls
across the bound on steps per launch."""
import numpy as np
import pytest

from oracle.oracle import Oracle
from paper_2512_06173_amd import workloads as W

pytestmark = pytest.mark.gpu


def mlk():
    from paper_2512_06173_amd import mlk as m
    return m


def ensemble(counts, seed, special=False):
    """counts[n]: emitters of n levels; special: one emitter with all levels degenerate,
    one without coupling and one with energies and couplings of 1e-170."""
    rng = np.random.default_rng(seed)
    nlev = np.concatenate([np.full(c, n, dtype=np.int32) for n, c in counts.items()])
    rng.shuffle(nlev)
    en, mop, rho = [], [], []
    for q, L in enumerate(nlev):
        e = np.sort(rng.uniform(0.0, 2.0, L))
        M = rng.standard_normal((L, L))
        M = 0.5 * (M + M.T)
        if special and q == 0:
            e[:] = 0.3
        if special and q == 1:
            M[:] = 0.0
        if special and q == 2:
            e, M = e * 1e-170, M * 1e-170
        v = rng.standard_normal(L) + 1j * rng.standard_normal(L)
        v /= np.linalg.norm(v)
        en.append(e)
        mop.append(M)
        rho.append(np.outer(v, v.conj()))
    n = len(nlev)
    return dict(nlev=nlev, energies=en, mop=mop, rho0=rho, dipole=rng.standard_normal((n, 3)),
                gphi=rng.uniform(0.0, 0.05, n), pos=rng.uniform(0.0, 16.0, (n, 3)),
                sigma=np.ones(n), gamma=np.ones(n))


@pytest.mark.parametrize("path", ["prescribed", "cavity"])
@pytest.mark.parametrize("counts", [{2: 1}, {6: 65}, {3: 64}, {2: 63, 3: 64, 4: 65, 5: 1, 6: 64},
                                    {4: 3, 6: 1}])
def test_level_counts_around_a_wavefront(counts, path):
    """Six steps, every state against the oracle.  Both sides are FP64 with a dozen
    operations of size one per entry and step: 6 x 6 levels x a few ulp stay below 1e-13."""
    m = ensemble(counts, 3 + sum(counts), special=sum(counts.values()) > 60)
    sim, ora = mlk().Simulation((16, 16, 16), bc=("periodic",) * 6), Oracle((16, 16, 16),
                                                                            bc=("periodic",) * 6)
    for o in (sim, ora):
        o.add_multilevel(**m)
    n = len(m["nlev"])
    if path == "cavity":
        for o in (sim, ora):
            o.set_cavity(0.25, 50.0, (0.3, -0.1), (0.0, 0.02))
        sim.step(6)
        ora.step(6)
    else:
        Et = 0.3 * np.random.default_rng(9).standard_normal((6, n, 3))
        sim.step_prescribed(Et)
        for q in range(6):
            ora.emitters_step_prescribed(Et[q])
    err = max(np.max(np.abs(sim.rho(q) - ora.rho(q))) for q in range(n))
    print(f"[levels] {path} {counts}: {err:.2e}", flush=True)
    # (the cavity's mean field adds its own rounding, summed over the ensemble)
    assert err <= (1e-13 if path == "prescribed" else 1e-12)


@pytest.mark.parametrize("steps", [1, 255, 256, 257, 515])
def test_steps_across_the_launch_bound(steps):
    """One call of many steps equals calls of one step each, bit for bit, recorded states
    and the last E~ and mu_dot among them (two-level and multilevel emitters)."""
    m = ensemble({2: 3, 5: 4}, 8)
    rng = np.random.default_rng(1)
    t = W.tls_ensemble(rng, 65, 0.0, 16.0, "superposition")
    sims = [mlk().Simulation((16, 16, 16), bc=("periodic",) * 6) for _ in range(2)]
    for s in sims:
        s.add_tls(t.pos, t.sigma, t.gamma, t.omega0, t.dipole, t.rho0)
        s.add_multilevel(**m)
    Et = 0.2 * rng.standard_normal((steps, 72, 3))
    a = sims[0].step_prescribed(Et, record=True)
    b = np.concatenate([sims[1].step_prescribed(Et[q:q + 1], record=True) for q in range(steps)])
    assert np.array_equal(a, b)
    assert all(np.array_equal(sims[0].rho(q), sims[1].rho(q)) for q in range(72))
    for x, y in zip(sims[0].emitter_io(), sims[1].emitter_io()):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("n_tls,n_ml", [(0, 0), (1, 0), (512, 0), (513, 3), (0, 65),
                                        (524288 + 300, 2), (3, 64 * 1024 + 70)])
def test_cavity_steps_do_not_depend_on_how_they_are_called(n_tls, n_ml):
    """Seven cavity steps in one call, in calls of one and with every step timed: mode,
    states, E~, mu_dot and populations bit for bit (block remainders, two-level ensembles
    walked with a stride, more partials than the blocks add up for themselves)."""
    rng = np.random.default_rng(5)
    t = W.tls_ensemble(rng, n_tls, 0.0, 16.0, "superposition") if n_tls else None
    m = ensemble({2: n_ml - n_ml // 3, 3: n_ml // 3}, 2) if n_ml else None
    out = []
    for mode in range(3):
        s = mlk().Simulation((16, 16, 16), bc=("periodic",) * 6)
        if t is not None:
            s.add_tls(t.pos, t.sigma, t.gamma, t.omega0, t.dipole, t.rho0)
        if m is not None:
            s.add_multilevel(**m)
        s.set_cavity(0.25, 1e4, (0.3, -0.1), (0.0, 0.02))
        s.record_populations(2)
        if mode == 2:
            s.set_timing(True)
        for k in [7] if mode != 1 else [1] * 7:
            s.step(k)
        s.sync()
        assert s.step_count == 7
        if mode == 2:
            assert s.phase_time("emitters")[1] == 7
        out.append([s.cavity(), s.populations(), *s.emitter_io(), s.checkpoint_save()])
        s.close()
    for o in out[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(out[0], o))
    assert np.any(out[0][0][:2] != (0.3, -0.1))
