"""The multilevel propagator over the sizes of H dt, from none to many turns a step, for every
level count."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [0.0, 1e-8, 0.3, 1.24, 1.26, 2.4, 2.6, 9.0, 60.0])
def test_unitary_step_against_eigenvectors(size):
    """One prescribed step with half the spread of H dt = size, against the exponential from
    numpy's eigenvectors.  Both sides turn phases up to size with relative rounding 2^-53
    in H, and take some tens of operations an entry: 64 (1 + size) 2^-53 on entries of at
    most one."""
    from paper_2512_06173_amd import mlk

    rng = np.random.default_rng(int(1e3 * size))
    sim = mlk.Simulation((16, 16, 16), bc=("periodic",) * 6)
    dt, en, mop, rho, nlev = sim.dt, [], [], [], []
    for q in range(70):
        n = 2 + q % 5
        H = rng.standard_normal((n, n))
        H = H + H.T
        ev = np.linalg.eigvalsh(H)
        H *= 2 * size / (dt * (ev[-1] - ev[0]))
        v = rng.standard_normal(n) + 1j * rng.standard_normal(n)
        v /= np.linalg.norm(v)
        nlev.append(n)
        en.append(np.diag(H).copy())
        mop.append(np.diag(np.diag(H)) - H)
        rho.append(np.outer(v, v.conj()))
    m = len(nlev)
    sim.add_multilevel(nlev=np.array(nlev, dtype=np.int32), energies=en, mop=mop, rho0=rho,
                       dipole=np.tile([1.0, 0.0, 0.0], (m, 1)), gphi=np.zeros(m),
                       pos=rng.uniform(0.0, 16.0, (m, 3)), sigma=np.ones(m), gamma=np.ones(m))
    sim.step_prescribed(np.tile([1.0, 0.0, 0.0], (1, m, 1)))
    err = 0.0
    for q in range(m):
        lam, Q = np.linalg.eigh(np.diag(en[q]) - mop[q])
        U = (Q * np.exp(-1j * lam * dt)) @ Q.T
        err = max(err, np.max(np.abs(sim.rho(q) - U @ rho[q] @ U.conj().T)))
    print(f"[norm] {size}: {err:.2e}", flush=True)
    assert err <= 64 * (1 + size) * 2.0 ** -53
