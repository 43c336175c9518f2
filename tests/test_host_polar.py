"""polar_rot, the Newton iteration behind the rigid update's rotation (eq. 6
for a well-conditioned matrix), compiled for the host from the kernels'
header and checked against numpy's SVD.  With C = U S V^T the rotation is
V diag(1, 1, sign det(V U^T)) U^T; its conditioning is 1 / (s2 + s3) of the
scaled matrix (at least 1/50 here), so 1e-13 leaves two digits over the
rounding of the entries.  Matrices it must leave to the SVD: reflections, flat
and singular ones, non-finite ones."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def polar(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("polar") / "polar_check")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-std=c++17", "-O2", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", os.path.join(HERE, "host", "polar_check.hip"), "-o", exe],
                   check=True, capture_output=True)

    def run(mats):
        text = "\n".join(" ".join(repr(float(x)) for x in np.asarray(A).ravel()) for A in mats) + "\n"
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True)
        rows = [np.array([float(v) for v in ln.split()]) for ln in out.stdout.strip().split("\n")]
        return [(int(r[0]), r[1:].reshape(3, 3)) for r in rows]
    return run


def _rot(rng):
    Q, _ = np.linalg.qr(rng.normal(size=(3, 3)))
    return Q * np.sign(np.linalg.det(Q))


def _kabsch(C):
    U, _, Vt = np.linalg.svd(C)
    return Vt.T @ np.diag([1.0, 1.0, np.sign(np.linalg.det(Vt.T @ U.T))]) @ U.T


def _matrix(rng, sv, scale=1.0):
    s = np.asarray(sv) / np.linalg.norm(sv) * np.sqrt(3.0)
    return scale * _rot(rng) @ np.diag(s) @ _rot(rng), float(np.prod(s))


def test_rotation_matches_svd(polar):
    rng = np.random.default_rng(4)
    mats, dets = [], []
    for sv in ([1, 1, 1], [1, 0.6, 0.4], [1, 0.36, 0.16], [1, 1, 0.02], [1, 0.1, 0.1], [3, 2, 1e-1], [1, 1, 0.0105]):
        for scale in (1.0, 1e-60, 1e60, 3.7e4):
            C, d = _matrix(rng, sv, scale)
            mats.append(C)
            dets.append(d)
    taken = 0
    for C, d, (ok, R) in zip(mats, dets, polar(mats)):
        if abs(d * 64 - 1) > 1e-9:
            assert ok == (d > 1.0 / 64), (C, d)
        if ok:
            taken += 1
            assert np.abs(R - _kabsch(C)).max() <= 1e-13
            assert np.abs(R @ R.T - np.eye(3)).max() <= 1e-14
    assert taken >= 20


def test_edge_of_the_accepted_range(polar):
    """Scaled determinants just above and below 1/64, the flattest accepted."""
    rng = np.random.default_rng(5)
    for f, want in ((1.001, 1), (0.999, 0)):
        # s1 = s2 = a, s3 = f / (64 a^2), normalised: solve for the norm sqrt(3)
        lo, hi = 1.0, 1.3
        for _ in range(200):
            a = 0.5 * (lo + hi)
            lo, hi = (a, hi) if 2 * a * a + (f / (64 * a * a)) ** 2 < 3 else (lo, a)
        C, d = _matrix(rng, [a, a, f / (64 * a * a)])
        assert abs(d * 64 - f) < 1e-6
        (ok, R), = polar([C])
        assert ok == want
        if ok:
            assert np.abs(R - _kabsch(C)).max() <= 1e-13


def test_left_to_the_svd(polar):
    rng = np.random.default_rng(6)
    refl = _matrix(rng, [1, 0.8, 0.5])[0] @ np.diag([1.0, 1.0, -1.0])
    flat = _matrix(rng, [1, 1, 1e-4])[0]
    line = np.outer([1, 2, 3], [3, 1, 1.0])
    bad = [refl, flat, line, np.zeros((3, 3)), np.full((3, 3), np.inf), np.full((3, 3), np.nan), np.eye(3) * 1e-140,
           np.eye(3) * 1e140]
    for C, (ok, _) in zip(bad, polar(bad)):
        assert ok == 0, C
