"""The wide tiles of the fused stress and LB on lattices large enough for them, with
remainders in every direction.

Debug mode: every LDS plane is NaN before a lattice plane is staged into it or the
stress evaluated into it, so a halo point that the kernels never write would come
out as NaN; results finite and bitwise those without the fills.  And the step
against the per-site one: FP64 to 300 roundings of the largest value after three
steps, as for the narrow tiles."""
import numpy as np
import pytest

from paper_0901_3293_amd import inputs as I
from tests.hlbtest import say

pytestmark = pytest.mark.gpu

SHAPES = [(126, 129, 97), (150, 94, 120), (126, 131, 128)]  # 64-site rows hanging over by 2, 42 and 2


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("coupling", ["force", "split"])
def test_wide_tiles_with_nan_filled_lds(prec, coupling):
    from paper_0901_3293_amd import hlb

    p = I.reduced(0.8, -0.3, 0.25)
    p.coupling = coupling
    eps = 2.0**-24 if prec == "fp32" else 2.0**-53
    for shape in SHAPES:
        Q = 0.4 * I.smooth_field(shape, 0.5, seed=3) + I.noise(shape, 1e-2, 4)
        out = []
        for sched, tz, nan in (("sites", 0, False), ("fused", 11, False), ("fused", 11, True), ("fused-tiled", 0, True)):
            say("case: wide tiles", shape, prec, coupling, sched, tz, nan)
            s = hlb.Solver(shape, prec, coupling=coupling)
            s.set_schedule(sched, tz)
            s.set_params(p)
            s.set_fields(Q)
            s.set_debug(nan_lds=nan)
            s.step(3)
            out.append([np.asarray(f) for f in s.fields()])
            s.close()
        for sites, plain, filled, tiled in zip(*out):
            assert np.array_equal(plain, filled)
            for other in (plain, tiled):
                assert np.isfinite(other).all() and np.abs(sites - other).max() <= 300 * eps * np.abs(sites).max(), shape
