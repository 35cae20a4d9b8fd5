"""The polarised-light texture at the ends of the range of its inputs: a
director within 1e-155 of the beam (tails of a localised texture in FP64; the
square of its in-plane part is below the smallest normal number), against the
oracle at the bar of the texture (1e-11 absolute), and retardances far past any
reduction of their angle (wavelengths down to the smallest numbers), where no
digit of the phase is left but every layer still is a rotation: images finite
and in [0, 1/2]."""
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


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_any_retardance_is_a_rotation(prec):
    Q = I.smooth_field((8, 7, 6), amp=0.3, seed=2)
    Q[:, 2] = 0.0  # an isotropic layer
    s = solver(Q, prec)
    for lam in (1e-6, 1e-9, 1e-12, 1e-16, 1e-18, 1e-25, 1e-100, 1e-300):
        say("case: optics, wavelength", lam, prec)
        img = s.optics(wavelengths=(lam, 18.0), weights=(0.5, 0.5))
        assert np.isfinite(img).all() and img.min() >= -1e-14 and img.max() <= 0.5 + 1e-14
    for lam in (1e-3, 1e-6):  # phases of 1e3 and 1e6: the texture's bar, 1e-11 at a wavelength of 16, grows with them
        kw = {"wavelengths": (lam,), "weights": (1.0,)}
        assert np.abs(s.optics(**kw) - OP.image(s.fields()[0], **kw)).max() <= 1e-11 * 16 / lam
    s = solver(np.zeros((5, 4, 4, 4)), prec)
    assert np.abs(s.optics(wavelengths=(1e-310,), weights=(1.0,))).max() <= 1e-14  # no retardance at all
