"""Disclination counts per plane without the fields (their own kernel, which cuts
every plane into chunks), against the oracle's (numpy eigh per site), exactly:
planes of one chunk, of several with a partial last one, and of chunks past 1024
sites (planes past 16384).  No site's eigenvalue lies within 1e-12 of a threshold."""
import numpy as np
import pytest

from oracle import order as O
from tests.hlbtest import say
from tests.test_gpu_order import H, solver, special_field  # noqa: F401  (H: a fixture)

pytestmark = pytest.mark.gpu

SHAPES = [(13, 7, 9), (4, 4, 4), (32, 32, 5), (33, 32, 4), (45, 37, 6), (64, 64, 5), (160, 130, 4), (20, 64, 400), (36, 36, 1030)]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_counts_per_plane(H, shape, prec):  # noqa: F811
    say("case: counts", shape, prec)
    s = solver(H, special_field(shape, seed=sum(shape)), prec)
    Qs = s.fields()[0]
    for threshold in (0.19, 0.12, 0.05, -0.01):
        q, _, below, _ = O.order(Qs, threshold)
        assert not (np.abs(q - threshold) <= 1e-12).any()
        per_z = O.defects_per_plane(below)
        res = s.order(threshold, fields=False)
        assert np.array_equal(res["per_z"], per_z) and res["n_defect"] == int(per_z.sum())
