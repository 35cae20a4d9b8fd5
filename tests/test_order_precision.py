"""The director of the fast eigen-solver (order.h, host build) against an
extended-precision one: no less precise than the Jacobi rotations that it stands
in for, from the smallest gap of the two largest eigenvalues that it takes
(about 0.0087 of the largest) to well separated ones.  Bar: the Jacobi sweeps'
own root mean square error on the same tensors."""
import numpy as np
import pytest

from tests.test_order_host import order_host, rotated  # noqa: F401  (order_host: a fixture)

LD = np.longdouble


def director_ld(q):
    """Eigenvector of the largest eigenvalue by Jacobi sweeps in extended precision."""
    a, b, c, e, f = q.astype(LD).T
    A = np.stack([np.stack([a, b, c], -1), np.stack([b, e, f], -1), np.stack([c, f, -a - e], -1)], -2)
    V = np.broadcast_to(np.eye(3, dtype=LD), A.shape).copy()
    for _ in range(8):
        for i, j in ((0, 1), (0, 2), (1, 2)):
            off = A[:, i, j]
            th = (A[:, j, j] - A[:, i, i]) / (2 * np.where(np.abs(off) > 1e-40, off, 1e-40))
            t = np.where(th >= 0, 1, -1) / (np.abs(th) + np.sqrt(th * th + 1))
            co = 1 / np.sqrt(t * t + 1)
            J = np.broadcast_to(np.eye(3, dtype=LD), A.shape).copy()
            J[:, i, i] = J[:, j, j] = co
            J[:, i, j], J[:, j, i] = t * co, -t * co
            A = np.einsum("nba,nbc,ncd->nad", J, A, J)
            V = np.einsum("nab,nbc->nac", V, J)
    n = np.arange(len(q))
    return V[n, :, np.argmax(A[:, range(3), range(3)], 1)]


@pytest.mark.skipif(np.finfo(LD).eps > 1e-18, reason="extended precision not available")
@pytest.mark.parametrize("gap", [0.0088, 0.01, 0.03, 0.1, 0.25, 0.4, 0.7])
def test_director_as_precise_as_by_jacobi(order_host, gap):  # noqa: F811
    rng = np.random.default_rng(int(1e4 * gap))
    g = gap * rng.uniform(1, 1.1, 4000)
    q = rotated(np.stack([0.5 + g, 0.5 - 0 * g, -1.0 - g], -1) * 0.3, rng)
    o, ref = order_host(q, 0.19), director_ld(q)
    assert np.all(o[:, 8] > 0)
    err = [np.sqrt((np.cross(d.astype(LD), ref) ** 2).sum(1)) for d in (o[:, 1:4], o[:, 5:8])]
    rms = [float(np.sqrt((e * e).mean())) for e in err]
    assert rms[0] <= rms[1], rms
