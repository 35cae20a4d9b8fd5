"""The per-site schedule on small lattices, whose sweeps run in pairs over
bricks of 16 x 4 x 2 sites, against the same schedule on a lattice large enough
for the single sweeps: a periodic cell repeated along each axis gives the
cell's step at every site.  The arithmetic per site is the same up to the
products that the compiler fuses: a site's update sums some hundred rounded
terms no larger than the field, so after three steps the two agree to 300
roundings of the largest value.  Cells at the edges of the bricks: smaller than a brick,
whole bricks, one site past them, and on either side of the 256 bricks (a CU
each) that still go in pairs; odd and even numbers of steps."""
import numpy as np
import pytest

from paper_0901_3293_amd import inputs as I
from tests.hlbtest import say

pytestmark = pytest.mark.gpu

CELLS = [(4, 4, 4), (5, 9, 7), (16, 8, 6), (17, 4, 5), (32, 32, 32), (33, 32, 32)]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("coupling", ["force", "split", "off"])
def test_brick_step_matches_the_single_sweeps(prec, coupling):
    from paper_0901_3293_amd import hlb

    eps = 2.0**-24 if prec == "fp32" else 2.0**-53
    for cell in CELLS:
        say("case: brick step", cell, prec, coupling)
        nx, ny, nz = cell
        rep = [1, 1, 1]
        while nx * ny * nz * np.prod(rep) <= 300000:  # far past 256 bricks
            rep[int(np.argmin([n * r for n, r in zip(cell, rep)]))] += 1
        p = I.reduced(0.8, -0.3, 0.25, flow=coupling != "off")
        p.coupling = "split" if coupling == "split" else "force"
        Q = 0.4 * I.smooth_field(cell, 0.5, seed=3) + I.noise(cell, 1e-2, 4)
        steps, out = 2 + cell[1] % 2, []
        for r in ([1, 1, 1], rep):
            s = hlb.Solver(tuple(n * k for n, k in zip(cell, r)), prec, coupling=coupling)
            s.set_params(p)
            s.set_fields(np.tile(Q, (1, r[2], r[1], r[0])))
            s.step(steps)
            out.append([np.asarray(f) for f in s.fields()])
            s.close()
        for name, a, b in zip(("Q", "u", "rho"), *out):
            whole = np.tile(a, (1,) * (a.ndim - 3) + (rep[2], rep[1], rep[0]))
            assert np.isfinite(a).all() and np.abs(whole - b).max() <= 300 * eps * np.abs(a).max(), (cell, name)
