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
    with np.errstate(over="ignore"):
        return np.array([np.argsort(_keys(P, q), kind="stable")[:k] for q in P[::step]], np.int32)


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


@pytest.mark.parametrize("n", [1, 40, 3000, 9000])
def test_ordinary_clouds(search, n):
    P = _surface(n, n)
    k, step = min(n, 24), max(1, n // 300)
    assert np.array_equal(search("knn", P, k, step).reshape(-1, k), _lists(P, k, step))
    rng = np.random.default_rng(4)
    Q = np.concatenate([P[::step] + rng.normal(size=P[::step].shape) * 0.05, rng.normal(size=(60, 3)) * 4]).astype(np.float32)
    for tau in (1e-3, 0.3, 1e18):
        assert np.array_equal(search("nn", P, len(Q), tau, Q), _nearest(P, Q, tau))
