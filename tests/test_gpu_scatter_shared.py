"""Scatter bins of more than 128 pairs, which the four wavefronts of a workgroup share: around
that limit, where quarters are ragged or empty, and with many times as many."""
import numpy as np
import pytest

from oracle.oracle import Oracle

pytestmark = pytest.mark.gpu

PEC, PER = ("pec",) * 6, ("periodic",) * 6
CASES = [((37, 23, 21), PEC), ((36, 12, 1), PER), ((9, 10, 11), PER)]


def mlk():
    from paper_2512_06173_amd import mlk as m
    return m


def run(make, shape, n, light=0, steps=1):
    """n emitters around one point and `light` ones all over the grid, driven alike."""
    rng = np.random.default_rng(n)
    s = make()
    s.set_eps(rng.uniform(1.0, 4.0, shape[::-1]))
    near = np.array([min(18.3, v / 2) for v in shape])
    pos = np.concatenate([near + rng.uniform(-0.3, 0.3, (n, 3)),
                          rng.uniform(np.minimum(4.0, near), np.maximum(np.array(shape) - 4.0, near),
                                      (light, 3))])
    m = n + light
    s.add_tls(pos, np.full(m, 1.0), rng.uniform(0.5, 1.5, m), np.full(m, 0.25),
              rng.uniform(0.5, 1.0, (m, 3)), np.tile([0.5, 0.1, 0.4], (m, 1)))
    s.step(steps)
    return s


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [127, 128, 129, 144, 145, 161, 257, 1000])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_shared_bins_against_the_oracle(case, n, precision):
    """One step from zero fields leaves E = -J / eps_r, every term of one sign: at most six
    roundings of a term and one per pair of a chunk-rounded quarter of the n, three in adding
    the quarters and E's own, of the largest |E|, with FP32 fields; FP64 holds 1e-13."""
    shape, bc = CASES[case]
    sim = run(lambda: mlk().Simulation(shape, precision=precision, bc=bc), shape, n)
    ora = run(lambda: Oracle(shape, bc=bc), shape, n)
    got, want = sim.fields()[:3], ora.fields()[:3]
    scale = max(np.max(np.abs(w)) for w in want)
    err = max(np.max(np.abs(a - b)) for a, b in zip(got, want)) / scale
    print(f"[shared] {shape} {precision} {n}: {err:.2e} of {scale:.2e}", flush=True)
    # (periodic axes shorter than a window take it in up to two pairs an axis)
    pairs = n * (1 if bc is PEC else 8) / 4 + 16
    assert scale > 0 and err <= (1e-13 if precision == "fp64" else (pairs + 10) * 2.0 ** -24)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_shared_and_other_bins_alone_and_in_a_batch(precision):
    """Workgroups of both kinds in one launch, with flux partials and sources behind them."""
    shape, out = (44, 40, 36), []
    for mode in ("alone", "again", "batch"):
        sims = []
        for _ in range(2 if mode == "batch" else 1):
            s = run(lambda: mlk().Simulation(shape, precision=precision), shape, 400, 300, 0)
            s.add_plane_source(2, 1, 1, 0.7, 0.3, 3.0, 2.0)
            s.add_flux_plane(0, 2)
            sims.append(s)
        if mode == "batch":
            b = mlk().Batch(sims)
            b.step(6)
            b.sync()
        else:
            sims[0].step(6)
        out += [s.fields() + [s.flux_series()] for s in sims]
        if mode == "batch":
            b.close()
        for s in sims:
            s.close()
    assert np.any(out[0][0])
    for o in out[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(out[0], o))


@pytest.mark.parametrize("n", [128, 1024, 1025, 2500, 12000])
def test_fp32_error_does_not_grow_with_the_emitters_around_a_cell(n):
    """A wavefront sums at most 256 pairs in FP32 before they are added up in FP64, four in one
    product: 64 roundings, each spread evenly over half a unit of the sum's last place (at most
    2^-24 of it), one of E and, far less over many terms, those of the terms.  The root mean
    square over the cells is then at most sqrt(66) 2^-24 / sqrt(3) = 2.8e-7 of the largest |E|,
    whatever n is.  (A sum of all pairs in FP32 passes that from some 4,000 on.)"""
    shape = (37, 23, 21)
    sim = run(lambda: mlk().Simulation(shape, precision="fp32"), shape, n)
    ora = run(lambda: Oracle(shape), shape, n)
    got, want = sim.fields()[:3], ora.fields()[:3]
    scale = max(np.max(np.abs(w)) for w in want)
    e = np.concatenate([(a - b)[np.abs(b) > 0.05 * scale] for a, b in zip(got, want)]) / scale
    rms = float(np.sqrt(np.mean(e ** 2)))
    print(f"[shared] fp32 {n}: rms {rms:.2e} over {e.size} cells", flush=True)
    assert rms <= np.sqrt(66 / 3) * 2.0 ** -24
