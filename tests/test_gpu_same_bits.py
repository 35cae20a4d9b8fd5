"""FP32 D3Q19 steps whose sweeps stand in for one another give the same bits: the
paired sweeps over bricks and the single ones (a periodic cell, and the cell repeated
along each axis to a lattice past the bricks), the fused stress and LB, on narrow and
on wide tiles, and the tiled stress against the per-site ones, and the tiled Q update,
at chunks of odd and of even numbers of planes, against the per-site predictor and
corrector.  The surrogate needs it: its jumps carry one rounding to 1e-4 within eight
cycles, and a run of it is repeated on whichever of these the lattice and the
autotuner pick."""
import numpy as np
import pytest

from paper_0901_3293_amd import inputs as I
from tests.hlbtest import say

pytestmark = pytest.mark.gpu

CELLS = [(4, 4, 4), (5, 9, 7), (16, 8, 6), (17, 4, 5), (32, 32, 32), (33, 32, 32)]
SHAPES = [(4, 4, 4), (17, 13, 9), (33, 25, 6), (65, 37, 12), (60, 44, 53), (96, 96, 96), (126, 129, 97), (128, 128, 128),
          (150, 100, 105)]


def run(shape, Q, coupling, schedule, steps):
    from paper_0901_3293_amd import hlb

    p = I.reduced(0.8, -0.3, 0.25, flow=coupling != "off")
    p.coupling = "split" if coupling == "split" else "force"
    s = hlb.Solver(shape, "fp32", coupling=p.coupling)
    s.set_schedule(*schedule)
    s.set_params(p)
    s.set_fields(Q)
    s.step(steps)
    out = [np.asarray(f) for f in s.fields()]
    s.close()
    return out


def field(shape):
    return 0.4 * I.smooth_field(shape, 0.5, seed=3) + I.noise(shape, 1e-2, 4)


@pytest.mark.parametrize("coupling", ["force", "split", "off"])
def test_bricks_and_single_sweeps(coupling):
    for cell in CELLS:
        say("case: bricks, same bits", cell, coupling)
        rep = [1, 1, 1]
        while np.prod(cell) * np.prod(rep) <= 300000:  # far past 256 bricks
            rep[int(np.argmin([n * r for n, r in zip(cell, rep)]))] += 1
        Q = field(cell)
        a = run(cell, Q, coupling, ("sites", 0), 5)
        b = run(tuple(n * r for n, r in zip(cell, rep)), np.tile(Q, (1, rep[2], rep[1], rep[0])), coupling, ("sites", 0), 5)
        for name, x, y in zip(("Q", "u", "rho"), a, b):
            whole = np.tile(x, (1,) * (x.ndim - 3) + (rep[2], rep[1], rep[0]))
            assert np.isfinite(x).all() and np.array_equal(whole, y), (cell, name)


@pytest.mark.parametrize("coupling", ["force", "split"])
def test_fused_and_per_site(coupling):
    for shape in SHAPES:
        Q = field(shape)
        a = run(shape, Q, coupling, ("sites", 0), 5)
        for tz in (1, 5, 16):
            say("case: fused, same bits", shape, coupling, tz)
            b = run(shape, Q, coupling, ("fused", tz), 5)
            for name, x, y in zip(("Q", "u", "rho"), a, b):
                assert np.isfinite(x).all() and np.array_equal(x, y), (shape, tz, name)


@pytest.mark.parametrize("coupling", ["force", "split", "off"])
def test_tiled_update_and_per_site(coupling):
    for shape in SHAPES:
        Q = field(shape)
        a = run(shape, Q, coupling, ("sites", 0), 6)
        for sched, tz in (("mixed", 1), ("mixed", 5), ("fused-tiled", 8), ("fused-tiled", 15), ("tiled", 6), ("tiled", 7)):
            if sched == "tiled" and coupling == "split":
                continue
            say("case: tiled update, same bits", shape, coupling, sched, tz)
            b = run(shape, Q, coupling, (sched, tz), 6)
            for name, x, y in zip(("Q", "u", "rho"), a, b):
                assert np.isfinite(x).all() and np.array_equal(x, y), (shape, sched, tz, name)
