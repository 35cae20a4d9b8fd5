"""The fused D3Q15 passes at the z-chunks that large lattices take, with one and
with several blocks after one another on a CU, whole tiles and remainders, against
the two sweeps of a small lattice: a periodic cell repeated along each axis gives
the cell's step at every site.  Bar as for the passes on mid-sized lattices: 300
roundings of the largest value after three steps."""
import numpy as np
import pytest

from paper_0901_3293_amd import inputs as I
from tests.hlbtest import say

pytestmark = pytest.mark.gpu

CELLS = [((10, 8, 10), (20, 25, 10)), ((16, 12, 6), (12, 16, 8)), ((13, 9, 7), (12, 15, 12)), ((10, 7, 9), (16, 20, 10))]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("coupling", ["force", "split"])
def test_fused_passes_on_large_lattices(prec, coupling):
    from paper_0901_3293_amd import hlb

    eps = 2.0**-24 if prec == "fp32" else 2.0**-53
    p = I.reduced(0.8, -0.3, 0.25)
    p.coupling, p.lb_model, p.tau = coupling, "d3q15", 5.0
    for cell, rep in CELLS:
        say("case: fused passes", cell, rep, prec, coupling)
        Q = 0.4 * I.smooth_field(cell, 0.5, seed=3) + I.noise(cell, 1e-2, 4)
        out = []
        for r in ((1, 1, 1), rep):
            s = hlb.Solver(tuple(n * k for n, k in zip(cell, r)), prec, coupling=coupling, lb_model="d3q15")
            s.set_params(p)
            s.set_fields(np.tile(Q, (1, r[2], r[1], r[0])))
            passes = [k for k, ms in s.step_timed(3).items() if k.startswith("k_pc") and ms > 0]
            assert passes == (["k_pc2"] if r == rep else ["k_pc1", "k_pc2"])
            out.append([np.asarray(f) for f in s.fields()])
            s.close()
        for name, a, b in zip(("Q", "u", "rho"), *out):
            whole = np.tile(a, (1,) * (a.ndim - 3) + (rep[2], rep[1], rep[0]))
            assert np.isfinite(a).all() and np.abs(whole - b).max() <= 300 * eps * np.abs(a).max(), (cell, name)
