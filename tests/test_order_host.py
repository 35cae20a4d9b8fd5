"""The eigen-solver of the order analysis (order.h, host build): the fast path
for a largest eigenvalue that stands clear of the middle one against the
Jacobi rotations it stands in for and against numpy's eigh, over random,
nearly degenerate, diagonal, uniaxial, scaled and non-finite tensors; and the
threshold test by minors against the eigenvalue it stands in for.

Bars: eigenvalue within 1e-14 of the spectral scale (the bar of the order
analysis); director parallel to 1e-9 and residual |Qd - qd| within 1e-13 of the
scale; the two decisions equal everywhere."""
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def order_host(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("order")
    exe = str(d / "order_host")
    subprocess.check_call([HIPCC, "-O2", "-std=c++17", os.path.join(HERE, "hostcheck", "order_host.cpp"), "-o", exe],
                          stderr=subprocess.DEVNULL)

    def run(q, threshold):
        np.concatenate([[len(q), threshold], np.ascontiguousarray(q, dtype=np.float64).ravel()]).tofile(d / "in")
        subprocess.check_call([exe, str(d / "in"), str(d / "out")])
        return np.fromfile(d / "out").reshape(-1, 10)

    return run


def full(q):
    return np.stack([np.stack([q[:, 0], q[:, 1], q[:, 2]], -1), np.stack([q[:, 1], q[:, 3], q[:, 4]], -1),
                     np.stack([q[:, 2], q[:, 4], -q[:, 0] - q[:, 3]], -1)], -2)


def five(T):
    return np.stack([T[:, 0, 0], T[:, 0, 1], T[:, 0, 2], T[:, 1, 1], T[:, 1, 2]], -1)


def rotated(lam, rng):
    R, _ = np.linalg.qr(rng.normal(size=(len(lam), 3, 3)))
    return five(R @ (lam[:, :, None] * np.eye(3)) @ R.transpose(0, 2, 1))


def tensors(kind, rng, n=20000):
    if kind == "random":
        return rng.normal(size=(n, 5)) * 0.2
    if kind == "top gap":  # from well separated down to equal in rounding
        g = 10.0 ** rng.uniform(-17, 0, n)
        return rotated(np.stack([0.5 + g, 0.5 - 0 * g, -1.0 - g], -1) * 0.3, rng)
    if kind == "gap at the limit of the fast path":
        g = 0.0087 * rng.uniform(0.8, 1.25, n)
        return rotated(np.stack([0.5 + g, 0.5 - 0 * g, -1.0 - g], -1), rng)
    if kind == "bottom gap":
        g = 10.0 ** rng.uniform(-17, 0, n)
        return rotated(np.stack([1.0 + 0 * g, -0.5 + g / 2, -0.5 - g / 2], -1) * 0.3, rng)
    if kind == "diagonal":
        lam = rng.normal(size=(n, 3))
        lam -= lam.mean(1, keepdims=True)
        return five(lam[:, :, None] * np.eye(3))
    if kind == "planar":  # the director in a coordinate plane
        q = rng.normal(size=(n, 5)) * 0.2
        q[:, [2, 4]] = 0
        return q
    if kind == "scales":
        return rng.normal(size=(n, 5)) * 10.0 ** rng.uniform(-30, 30, (n, 1))
    q = rng.choice([0.0, 0.1, -0.2, 1e-300], size=(n, 5))
    return q


KINDS = ["random", "top gap", "gap at the limit of the fast path", "bottom gap", "diagonal", "planar", "scales", "zeros"]


@pytest.mark.parametrize("kind", KINDS)
def test_order_site_against_jacobi_and_eigh(order_host, kind):
    rng = np.random.default_rng(KINDS.index(kind))
    q = tensors(kind, rng)
    o = order_host(q, 0.19)
    T = full(q)
    w, v = np.linalg.eigh(T)
    scale = np.abs(w).max(1)
    ok = scale > 1e-150  # the squared norm of smaller ones underflows on both paths
    lam, d, jl, jd, fast = o[:, 0], o[:, 1:4], o[:, 4], o[:, 5:8], o[:, 8] > 0
    if kind in ("random", "bottom gap", "planar"):
        assert fast.mean() > 0.99
    assert np.all(np.abs(lam - w[:, 2])[ok] <= 1e-14 * scale[ok])
    assert np.all(np.abs(lam - jl)[ok] <= 1e-14 * scale[ok])
    assert np.abs((d * d).sum(1) - 1).max() <= 1e-14
    r = np.linalg.norm(np.einsum("nab,nb->na", T, d) - lam[:, None] * d, axis=1)
    assert np.all(r[ok] <= 1e-13 * scale[ok])
    sep = ok & (w[:, 2] - w[:, 1] > 1e-6 * scale)
    assert np.all(np.abs(np.abs((d * v[:, :, 2]).sum(1)) - 1)[sep] <= 1e-9)
    last = np.where(d[:, 2] != 0, d[:, 2], np.where(d[:, 1] != 0, d[:, 1], d[:, 0]))
    assert np.all(last > 0)
    # an axis that the tensor leaves uncoupled: the director lies along it or has no component there
    for axis, off in ((0, [1, 2]), (1, [1, 4]), (2, [2, 4])):
        u = sep & (q[:, off] == 0).all(1)
        for e in (d, jd):
            assert np.all((e[u, axis] == 0) | (np.abs(np.delete(e[u], axis, 1)).max(1, initial=0) == 0))


@pytest.mark.parametrize("threshold", [0.19, 0.0, -0.1, 0.05, 1e9])
def test_threshold_by_minors(order_host, threshold):
    rng = np.random.default_rng(11)
    q = np.concatenate([tensors(k, rng, 4000) for k in KINDS])
    # eigenvalues within a few roundings of the threshold, and just clear of it
    g = np.concatenate([rng.uniform(-4e-16, 4e-16, 2000), rng.uniform(-1e-11, 1e-11, 2000)])
    t = abs(threshold) + 0.01
    near = rotated(np.stack([threshold + g * t, -threshold / 2 - t + 0 * g, -threshold / 2 + t - g * t], -1), rng)
    bad = np.array([[np.nan] * 5, [np.inf, 0, 0, 0, 0], [0, np.inf, 0, 0, 0], [0.1, 0, np.nan, 0, 0]])
    q = np.concatenate([q, near, bad])
    o = order_host(q, threshold)
    with np.errstate(invalid="ignore"):
        assert np.array_equal(o[:, 9] > 0, o[:, 0] < threshold)
        assert np.array_equal(np.isnan(o[:, 0]), np.isnan(o[:, 4]))
