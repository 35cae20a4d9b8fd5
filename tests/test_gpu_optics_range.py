"""The polarised-light texture at the ends of the range of its inputs: a
director within 1e-155 of the beam (tails of a localised texture in FP64; the
square of its in-plane part is below the smallest normal number), against the
oracle at the bar of the texture (1e-11 absolute)."""
import numpy as np
import pytest

from oracle import optics as OP
from paper_0901_3293_amd import inputs as I
from tests.hlbtest import say

pytestmark = pytest.mark.gpu


def solver(Q, prec):
    from paper_0901_3293_amd import hlb

    nz, ny, nx = Q.shape[1:]
    s = hlb.Solver((nx, ny, nz), prec)
    s.set_params(I.PhysParams(K=0.02, q0=0.3))
    s.set_fields(Q, None, None)
    return s


@pytest.mark.parametrize("tilt", [1e-140, 1e-152, 1e-154, 1e-155, 1e-157, 1e-161, 1e-165])
def test_director_along_the_beam_but_for_a_tail(tilt):
    say("case: optics, director along the beam but for", tilt)
    rng = np.random.default_rng(5)
    Q = I.smooth_field((8, 7, 6), amp=0.3, seed=2)  # [c][z][y][x]
    # half of the sites: uniaxial along z, tilted by `tilt` in a random direction
    along = rng.random(Q.shape[1:]) < 0.5
    for k, v in enumerate((-0.1, 0.0, None, -0.1, None)):
        Q[k][along] = rng.uniform(0.3, 1.0, along.sum()) * tilt if v is None else v
    s = solver(Q, "fp64")
    img, ref = s.optics(), OP.image(s.fields()[0])
    assert np.isfinite(img).all() and np.abs(img - ref).max() <= 1e-11
