"""An adjoint call leaves the device memory that it found free: nothing is kept for the next
call, below and above a GiB of checkpoints, and the gradients do not depend on what ran before."""
import numpy as np
import pytest

from paper_2512_06173_amd import workloads as W

pytestmark = pytest.mark.gpu


def mlk():
    from paper_2512_06173_amd import mlk as m
    return m


def make(n, precision, sweep="fused"):
    s = mlk().Simulation((n, n, n), precision=precision, bc=("cpml",) * 6, cpml=(6,) * 6,
                         sweep=sweep)
    t = W.tls_ensemble(np.random.default_rng(1), 12, n / 2 - 5.0, n / 2 + 5.0, "superposition")
    s.add_tls(t.pos, t.sigma, t.gamma, t.omega0, t.dipole, t.rho0)
    s.add_flux_plane(2, n - 9)
    return s


def call(s, n, steps, every):
    h = n // 2
    return s.adjoint("flux", steps, ((h - 4,) * 3, (h + 4,) * 3), checkpoint_every=every)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,steps,every", [(40, 9, 4), (40, 12, 1), (96, 40, 1)])
def test_nothing_is_kept(n, steps, every, precision):
    import torch
    warm = make(40, precision)  # modules, streams and the like
    call(warm, 40, 2, 1)
    with make(n, precision) as s:
        s.step(steps + 2)  # room in the series
        s.sync()
        free = torch.cuda.mem_get_info()[0]
        print(f"[adjoint memory] {n} {steps} {every} {precision}", flush=True)
        a = call(s, n, steps, every)
        assert torch.cuda.mem_get_info()[0] == free
        call(s, n, steps + 1, every + 1)  # another shape
        b = call(s, n, steps, every)
        assert torch.cuda.mem_get_info()[0] == free
        assert a[0] == b[0] and all(np.array_equal(x, y) for x, y in zip(a[1:], b[1:]))
    warm.close()
