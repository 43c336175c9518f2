"""The bounds of the neighbour search's grid (csrc/grid_geom.h), compiled for
the host into a serial search in the kernels' order of places, against brute
force: neighbour lists and nearest points exactly (FP32 keys, ties by index)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def search(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("grid") / "grid_check")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-std=c++17", "-O2", "-ffp-contract=off", "-Xclang",
                    "-target-feature", "-Xclang", "-packed-fp32-ops", os.path.join(HERE, "host", "grid_check.hip"),
                    "-o", exe], check=True, capture_output=True)

    def run(what, P, arg, last, Q=None):
        data = P.tobytes() + (b"" if Q is None else Q.tobytes())
        out = subprocess.run([exe, what, str(len(P)), str(arg), str(last)], input=data, capture_output=True,
                             timeout=100)
        assert out.returncode == 0, out.stderr
        return np.frombuffer(out.stdout, np.int32)
    return run


def _keys(P, q):
    d = P - q
    return (d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2]


def _lists(P, k, step):
    """-1 where fewer than k points have a finite key."""
    out = []
    with np.errstate(over="ignore"):
        for q in P[::step]:
            d = _keys(P, q)
            i = np.argsort(d, kind="stable")[:k]
            out.append(np.where(np.isfinite(d[i]), i, -1))
    return np.array(out, np.int32)


def _nearest(P, Q, tau):
    with np.errstate(over="ignore"):
        keys = [_keys(P, q) for q in Q]
    best = np.array([d.argmin() for d in keys], np.int32)
    return np.where(np.array([d.min() for d in keys]) <= np.float32(tau) * np.float32(tau), best, -1)


def _surface(n, seed):
    rng = np.random.default_rng(seed)
    u = rng.normal(size=(n, 3))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    return (u * [1.0, 0.7, 0.4] + rng.normal(size=(n, 3)) * 0.002).astype(np.float32)


def _long(kind, n, axis, seed):
    """A pipe 1 000 long of radius 0.5, or a strip 300 x 1, along an axis."""
    rng = np.random.default_rng(seed)
    if kind == "pipe":
        f = rng.uniform(0, 2 * np.pi, n)
        P = np.stack([rng.uniform(0, 1000, n), 0.5 * np.cos(f), 0.5 * np.sin(f)], 1)
    else:
        P = np.stack([rng.uniform(0, 300, n), rng.uniform(0, 1, n), rng.normal(size=n) * 1e-3], 1)
    return np.roll(P, axis, axis=1).astype(np.float32)


def _cloud(kind, axis, side):
    if kind == "stray point":
        P = _surface(20000, 1)
        P[17] = 0
        P[17, axis] = side * 500
        return P
    return _long(kind, 6000, axis, 2)


# Grids with nearly all of their cells along one axis.
LONG = [("stray point", a, s) for a in range(3) for s in (1, -1)] + \
       [(kind, a, 1) for kind in ("pipe", "strip") for a in range(3)]


@pytest.mark.parametrize("kind,axis,side", LONG)
def test_lists_of_clouds_longer_than_the_grid(search, kind, axis, side):
    P = _cloud(kind, axis, side)
    k, step = 16, len(P) // 250
    assert np.array_equal(search("knn", P, k, step).reshape(-1, k), _lists(P, k, step))


@pytest.mark.parametrize("kind,axis,side", LONG)
@pytest.mark.parametrize("tau", [0.05, 1e18])
def test_nearest_points_of_clouds_longer_than_the_grid(search, kind, axis, side, tau):
    P = _cloud(kind, axis, side)
    rng = np.random.default_rng(3)
    near = P[::len(P) // 200]
    Q = np.concatenate([near + rng.normal(size=near.shape) * 0.01, near[::5] * 1.02,
                        rng.normal(size=(40, 3)) * 400]).astype(np.float32)
    assert np.array_equal(search("nn", P, len(Q), tau, Q), _nearest(P, Q, tau))


@pytest.mark.parametrize("n", [1, 40, 3000, 9000])
def test_ordinary_clouds(search, n):
    P = _surface(n, n)
    k, step = min(n, 24), max(1, n // 300)
    assert np.array_equal(search("knn", P, k, step).reshape(-1, k), _lists(P, k, step))
    rng = np.random.default_rng(4)
    Q = np.concatenate([P[::step] + rng.normal(size=P[::step].shape) * 0.05, rng.normal(size=(60, 3)) * 4]).astype(np.float32)
    for tau in (1e-3, 0.3, 1e18):
        assert np.array_equal(search("nn", P, len(Q), tau, Q), _nearest(P, Q, tau))


@pytest.mark.parametrize("scale", [1e-38, 1e-30, 1e-24, 1e-22, 1e-20, 1e-18, 1e-16, 1e-10, 1e10, 1e17, 1e18, 1e25, 1e35])
def test_clouds_of_any_scale(search, scale):
    """Keys that underflow (many are 0, and ties go by index) and overflow."""
    P = np.concatenate([_surface(3000, 5), np.float32([[3, 0, 0], [0, 30, 0], [0, 0, -300]])]) * np.float32(scale)
    for k in (5, 24):
        assert np.array_equal(search("knn", P, k, 10).reshape(-1, k), _lists(P, k, 10))
    rng = np.random.default_rng(6)
    with np.errstate(over="ignore"):
        Q = np.concatenate([P[::10] * np.float32(1.01), rng.normal(size=(60, 3)).astype(np.float32) * np.float32(scale)])
    Q = Q[np.isfinite(Q).all(1)]
    assert np.array_equal(search("nn", P, len(Q), 1.8e19, Q), _nearest(P, Q, 1.8e19))


@pytest.mark.parametrize("e", [3, 8, 16, 18, 18.6, 18.9, 19, 20, 38])
def test_nearest_points_of_queries_far_away(search, e):
    """Up to where every key overflows (no nearest point)."""
    P = _surface(3000, 5)
    u = np.random.default_rng(7).normal(size=(100, 3))
    Q = (u / np.linalg.norm(u, axis=1, keepdims=True) * 10.0 ** e).astype(np.float32)
    with np.errstate(over="ignore"):
        keys = [_keys(P, q) for q in Q]
    want = [d.argmin() if np.isfinite(d.min()) else -1 for d in keys]
    assert np.array_equal(search("nn", P, len(Q), np.inf, Q), want)
