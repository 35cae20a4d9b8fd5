"""The free-energy profile f(z) at the sizes where its planes are cut into chunks or
stay whole: a periodic cell repeated along z, every plane against the oracle's plane
sum of the cell.  Bars: 1e-12 in FP64, 1e-5 in FP32 (those of the profile) of the
plane's sum of magnitudes."""
import numpy as np
import pytest

from paper_0901_3293_amd import inputs as I
from tests.hlbtest import oracle_params, say

pytestmark = pytest.mark.gpu

# planes of 1280 and 1350 sites: 378 in two chunks, 384 whole; 4096 and 4180 sites: four and five chunks of any
# number; one chunk; past 16 chunks of 1024 sites
CASES = [((64, 20, 6), 63), ((64, 20, 6), 64), ((45, 30, 6), 64), ((64, 64, 4), 100), ((44, 95, 4), 98), ((16, 12, 5), 2),
         ((130, 131, 4), 1)]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_profile_in_chunks(orc, prec):
    from paper_0901_3293_amd import hlb

    p = I.reduced(0.8, -0.3, 0.25)
    for cell, rep in CASES:
        say("case: f(z) in chunks", cell, rep, prec)
        Q = 0.4 * I.smooth_field(cell, 0.5, seed=3) + I.noise(cell, 1e-2, 4)
        Qs = Q if prec == "fp64" else Q.astype(np.float32).astype(np.float64)
        _, f, _ = orc.chem(oracle_params(orc, p), orc.q5_to_q9(Qs))
        ref = np.tile(np.array([orc.psum(f[z]) for z in range(cell[2])]), rep)
        s = hlb.Solver((cell[0], cell[1], cell[2] * rep), prec)
        s.set_params(p)
        s.set_fields(np.tile(Q, (1, rep, 1, 1)))
        fz = s.fz()
        s.close()
        scale = np.abs(f).sum(axis=(1, 2)).max()
        assert np.abs(fz - ref).max() <= (1e-12 if prec == "fp64" else 1e-5) * scale, (cell, rep)
