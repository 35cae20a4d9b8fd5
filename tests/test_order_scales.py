"""The threshold test by minors (order.h, host build) against the eigenvalue it
stands in for, on tensors and thresholds of any common scale: also where the
cube of the scale underflows or overflows."""
import numpy as np
import pytest

from tests.test_order_host import order_host  # noqa: F401  (a fixture)


@pytest.mark.parametrize("scale", [-160, -150, -120, -109, -108, -107, -104, -91, -90, -89, -30, 30, 89, 90, 91, 102, 103,
                                   104, 150])
def test_threshold_by_minors_at_any_scale(order_host, scale):  # noqa: F811
    rng = np.random.default_rng(1000 + scale)
    for threshold in (0.3, 0.0, -0.2):
        q = rng.normal(size=(20000, 5)) * 10.0**scale
        o = order_host(q, threshold * 10.0**scale)
        assert np.array_equal(o[:, 9] > 0, o[:, 0] < threshold * 10.0**scale)
