"""Soft sources of one component that share cells: two pulses on one plane, planes that cross,
a point on a plane and on their crossing, and two points in one cell.  Against the oracle,
whether the sources have a launch of their own or ride in the scatter's, alone and in a batch."""
import numpy as np
import pytest

from oracle.oracle import Oracle
from paper_2512_06173_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPE = (26, 22, 24)
# plane (axis, index) or point (i, j, k) of component 1; the emitters' windows reach neither
# (folded) or all of them (not)
SETS = [[(2, 3), (2, 3)], [(2, 3), (0, 20), (20, 5, 3)], [(20, 5, 3), (2, 3), (0, 20)],
        [(21, 4, 3), (21, 4, 3), (2, 2)],
        [(2, 3), (0, 20), (2, 3), (20, 5, 3), (20, 5, 9), (0, 20), (20, 5, 3), (2, 3)]]


def mlk():
    from paper_2512_06173_amd import mlk as m
    return m


def fill(s, which, near):
    rng = np.random.default_rng(5)
    s.set_eps(rng.uniform(1.0, 3.0, SHAPE[::-1]))
    lo, hi = ((5, 5, 6), (21, 17, 18)) if near else ((6, 8, 12), (12, 14, 18))
    pos = rng.uniform(lo, hi, (25, 3))
    s.add_tls(pos, np.ones(25), np.ones(25), np.full(25, 0.25),
              np.tile([0.3, 0.2, -0.4], (25, 1)), np.tile([0.5, 0.1, 0.4], (25, 1)))
    for q, v in enumerate(SETS[which]):
        wave = (0.5 + 0.3 * q, 0.3 + 0.02 * q, 4.0, 3.0 + q)
        if len(v) == 2:
            s.add_plane_source(v[0], v[1], 1, *wave)
        else:
            s.add_point_source(1, v, *wave)


def rel(a, b):
    a, b = (np.concatenate([np.ravel(x) for x in v]) for v in (a, b))
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("near", [False, True])
@pytest.mark.parametrize("which", range(len(SETS)))
def test_overlapping_sources_against_the_oracle(which, near, precision):
    """The parity bounds: 1e-12 of the fields with FP64, 1e-4 with FP32 (a lost update is a
    whole source's share); each way of launching the sources gives the same bits."""
    print(f"[sources] set {which} near={near} {precision}", flush=True)
    ora = Oracle(SHAPE)
    fill(ora, which, near)
    ora.step(12)
    tol = 1e-12 if precision == "fp64" else 1e-4
    first = None
    for mode in ("alone", "timed", "batch", "plain"):
        sims = [mlk().Simulation(SHAPE, precision=precision,
                                 sweep="plain" if mode == "plain" else "fused")
                for _ in range(3 if mode == "batch" else 1)]
        for s in sims:
            fill(s, which, near)
            if mode == "timed":
                s.set_timing(["sources"])
        if mode == "batch":
            b = mlk().Batch(sims)
            b.step(12)
            b.sync()
        else:
            sims[0].step(12)
        got = [s.fields() for s in sims]
        for f in got:
            assert rel(f, ora.fields()) <= tol
            if mode != "plain":
                first = first or f
                assert all(np.array_equal(x, y) for x, y in zip(first, f))
        if mode == "batch":
            b.close()
        for s in sims:
            s.close()
