"""The tiling that a new simulation starts from, at each line of its rule: the fields are
those of the plain sweep bit for bit, alone and as an untuned member of a batch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PEC, CPML, Z = ("pec",) * 6, ("cpml",) * 6, ("periodic",) * 4 + ("cpml",) * 2


def mlk():
    from paper_2512_06173_amd import mlk as m
    return m


# shape, boundaries, CPML cells, FP32 rule: (tile width, ty, kz, layers)
CASES = [((32, 32, 32), CPML, 6, (32, 4, 1, 1)),      # less than one round of single planes
         ((64, 33, 150), CPML, 5, (64, 8, 2, 1)),     # tall tiles, two planes
         ((96, 64, 80), CPML, 8, (32, 16, 2, 1)),     # half tiles
         ((96, 64, 80), PEC, 0, (32, 16, 2, 1)),      # a higher round without layers
         ((36, 20, 18), CPML, 5, (64, 4, 1, 1)),      # ragged rows
         ((200, 140, 90), CPML, 8, (64, 8, 13, 1)),  # ragged, chunks of up to 16 planes
         ((200, 200, 100), CPML, 8, (64, 8, 8, 1)),   # ragged, more than 16: short chunks
         ((320, 300, 70), CPML, 8, (64, 16, 32, 1)),  # several rounds: 32 planes
         ((96, 12, 1), ("periodic",) * 6, 0, (32, 4, 1, 1)), ((5, 4, 9), PEC, 0, (64, 4, 1, 1)),
         ((128, 4, 40), Z, 7, (64, 4, 1, 1))]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_default_tiling(case, precision):
    shape, bc, npml, rule = CASES[case]
    cp = tuple(npml if b == "cpml" else 0 for b in bc)
    rng = np.random.default_rng(case)
    start = [rng.standard_normal(shape[::-1]) for _ in range(6)]
    for f in start:  # walls hold no field
        for axis in range(3):
            if bc[2 * (2 - axis)] != "periodic":
                for end in (0, -1):
                    f[(slice(None),) * axis + (end,)] = 0.0

    def sim(**kw):
        s = mlk().Simulation(shape, precision=precision, bc=bc, cpml=cp, **kw)
        for c in range(6):
            s.set_field(c, start[c])
        return s

    plain, alone, member = sim(sweep="plain"), sim(), sim()
    got = (alone.tile_width(), *alone.tuning()[:2], alone.sweep_layers())
    print(f"[tiling] {shape} {precision} {got}", flush=True)
    if precision == "fp32":
        assert got == rule
    else:
        assert got[:2] == (64, 4) and got[2] <= 8 and got[3] == 0
    plain.step(6)
    alone.step(6)
    b = mlk().Batch([member])
    assert member.tile_width() == 64 and member.tuning()[0] == 4
    b.step(6)
    b.close()
    member.step(4)
    alone.step(4)
    plain.step(4)
    for x, y, z in zip(plain.fields(), alone.fields(), member.fields()):
        assert np.array_equal(x, y) and np.array_equal(x, z)
