"""The scatter with FP32 fields and amplitudes beyond FP32: what a cell receives is the amplitude
times a weight, which FP32 may hold all the same, and cells that no window reaches are left alone."""
import numpy as np
import pytest

from oracle.oracle import Oracle

pytestmark = pytest.mark.gpu


def mlk():
    from paper_2512_06173_amd import mlk as m
    return m


def run(make, amps, sigma):
    """One step from zero fields of emitters along one row of 16-cell bins."""
    s = make()
    n = len(amps)
    pos = np.column_stack([4.3 + 9.0 * np.arange(n), np.full(n, 6.2), np.full(n, 6.1)])
    # mu_dot = -2 omega0 Im rho01 d, and the amplitude dt gamma mu_dot = -0.1 d
    s.add_tls(pos, np.full(n, sigma), np.ones(n), np.full(n, 0.25),
              np.outer(-10.0 * np.asarray(amps), [1.0, -0.5, 0.25]), np.tile([0.5, 0.1, 0.4], (n, 1)))
    s.step(1)
    return [np.asarray(f) for f in s.fields()[:3]]


@pytest.mark.parametrize("sigma", [0.6, 1.0, 1.05])
def test_amplitudes_beyond_fp32(sigma):
    shape = (32, 13, 13)
    amps = [1.0e37, 7.0e38, 3.0e36]
    got = run(lambda: mlk().Simulation(shape, precision="fp32"), amps, sigma)
    want = run(lambda: Oracle(shape), amps, sigma)
    scale = max(np.max(np.abs(w)) for w in want)
    assert 3e37 < scale < 3.4e38  # FP32 holds every cell
    for g, w in zip(got, want):
        # six roundings of a term and one each of the sum over at most three and of E
        assert np.max(np.abs(g - w)) <= 10 * 2.0 ** -24 * scale
        assert np.array_equal(g == 0.0, w.astype(np.float32) == 0.0)


@pytest.mark.parametrize("big", [1e60, 1e300])
def test_amplitudes_far_beyond_fp32_stay_in_their_window(big):
    shape = (32, 13, 13)
    got = run(lambda: mlk().Simulation(shape, precision="fp32"), [2.0, big, 3.0], 1.0)
    want = run(lambda: Oracle(shape), [2.0, 0.0, 3.0], 1.0)
    for g, w in zip(got, want):
        assert not np.any(np.isnan(g)) and np.any(np.isinf(g))
        assert np.max(np.abs(g[..., :9] - w[..., :9])) <= 10 * 2.0 ** -24 * np.max(np.abs(w))
        assert np.max(np.abs(g[..., 18:] - w[..., 18:])) <= 10 * 2.0 ** -24 * np.max(np.abs(w))
