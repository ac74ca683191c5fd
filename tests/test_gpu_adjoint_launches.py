"""The one launch of the fused transposed sweep (box, z-face slabs, E pass of the shell) at the
edges of its cuts: x layers that keep the box off the first columns (the E pass then has its
own launch), layers through the whole depth, chunks of many lengths, no layers."""
import numpy as np
import pytest

from paper_2512_06173_amd import workloads as W

pytestmark = pytest.mark.gpu


def mlk():
    from paper_2512_06173_amd import mlk as m
    return m


PZ = ("periodic",) * 4 + ("cpml",) * 2
CASES = [((70, 26, 40), ("cpml",) * 6, (8, 8, 5, 5, 5, 5), True),
         ((64, 24, 15), PZ, (0, 0, 0, 0, 7, 7), False),
         ((64, 20, 12), PZ, (0, 0, 0, 0, 6, 6), False),
         ((96, 20, 300), PZ, (0, 0, 0, 0, 6, 9), True),
         ((40, 70, 30), ("cpml",) * 6, (5,) * 6, True),
         ((33, 18, 20), ("pec",) * 6, (0,) * 6, True)]


def rel(a, b):
    return np.linalg.norm(np.ravel(a) - np.ravel(b)) / np.linalg.norm(np.ravel(b))


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_fused_adjoint_matches_plain(case, precision):
    """Gradients against those of the whole-grid transposed sweep.  Both round each cell's
    update in its own order: 2e-5 with FP32 fields over 30 steps, 1e-12 with FP64."""
    shape, bc, cpml, emitters = CASES[case]
    rng = np.random.default_rng(case)
    mid = np.array(shape) / 2
    tls = None
    if emitters:
        tls = W.TLSSet(pos=mid + rng.uniform(-1, 1, (4, 3)), sigma=np.full(4, 0.8),
                       gamma=np.ones(4), omega0=rng.uniform(0.45, 0.55, 4),
                       dipole=0.6 * rng.standard_normal((4, 3)),
                       rho0=np.tile([0.5, 0.5, 0.0], (4, 1)))
    src = tuple(int(v) for v in mid - 1)
    w = W.Workload(name="adj_cuts", shape=shape, bc=bc, cpml=cpml,
                   eps=rng.uniform(1.0, 2.0, shape[::-1]), tls=tls,
                   point_sources=[W.PointSource(1, src, 1.0, 0.5, 2.0, 6.0)],
                   flux=(2, shape[2] // 2 + 2), steps=30, precision=precision)
    box = (tuple(m - 3 for m in src), tuple(m + 3 for m in src))
    res = []
    for sweep in ("fused", "plain"):
        sim = mlk().from_workload(w, sweep=sweep)
        res.append(sim.adjoint("flux", w.steps, box, checkpoint_every=15))
    (fv, fge, fgd), (pv, pge, pgd) = res
    tol = 2e-5 if precision == "fp32" else 1e-12
    print(f"[adjoint cuts] {shape} {precision}: value {abs(fv - pv) / abs(pv):.2e}, eps "
          f"{rel(fge, pge):.2e}", flush=True)
    assert abs(fv - pv) <= tol * abs(pv) and rel(fge, pge) <= tol
    if emitters:
        assert rel(fgd, pgd) <= tol


def test_adjoint_calls_of_changing_shape():
    """The device blocks kept between calls: calls with other steps, checkpoints and boxes in
    between (more and less of everything) leave a call's result as it was, bit for bit."""
    shape = (40, 30, 28)
    rng = np.random.default_rng(3)
    tls = W.TLSSet(pos=np.array(shape) / 2 + rng.uniform(-1, 1, (4, 3)), sigma=np.full(4, 0.8),
                   gamma=np.ones(4), omega0=rng.uniform(0.45, 0.55, 4),
                   dipole=0.6 * rng.standard_normal((4, 3)), rho0=np.tile([0.5, 0.5, 0.0], (4, 1)))
    w = W.Workload(name="adj_shapes", shape=shape, bc=("cpml",) * 6, cpml=(5,) * 6,
                   eps=rng.uniform(1.0, 2.0, shape[::-1]), tls=tls,
                   point_sources=[W.PointSource(1, (19, 14, 13), 1.0, 0.5, 2.0, 6.0)],
                   flux=(2, 16), steps=20, precision="fp32")
    sim = mlk().from_workload(w, sweep="fused")
    box = ((16, 11, 10), (22, 17, 16))
    calls = [(20, box, 8), (20, box, 8), (31, ((10, 10, 10), (28, 20, 20)), 5), (20, box, 8),
             (3, ((16, 11, 10), (17, 12, 11)), 3), (20, box, 8)]
    res = [sim.adjoint("flux", n, b, checkpoint_every=k) for n, b, k in calls]
    for q in (1, 3, 5):
        assert res[q][0] == res[0][0]
        assert all(np.array_equal(x, y) for x, y in zip(res[q][1:], res[0][1:]))
