"""The one-launch iteration loop of flags bit 3 (points in registers, blocks
exchanging their partial wrenches) against the per-iteration kernels, which
the library runs by itself when the loop gives up waiting: a poll limit of 1
(SGR_LOOP_SPINS, read when a context is made) makes a loop of several blocks
give up, and the registration starts again from its initial pose.  Both pose
the same float32 points and add the same float64 terms in another order:
1e-10 in every pose entry and 1e-10 relative in the statistics leaves four
digits over that rounding through the iterations run here."""
import os

import numpy as np
import pytest
import torch

from synth import config1, random_pair, super_fibonacci_rotations

pytestmark = pytest.mark.gpu

SUMS = 8


@pytest.fixture(scope="module")
def sg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_01061_amd as sg
    return sg


@pytest.fixture(scope="module")
def both(sg):
    """(a context whose loop runs, a context whose loop gives up)."""
    loop = sg.Context(0)
    os.environ["SGR_LOOP_SPINS"] = "1"
    try:
        steps = sg.Context(0)
    finally:
        del os.environ["SGR_LOOP_SPINS"]
    yield loop, steps
    loop.close()
    steps.close()


def _close(a, b, tol=1e-10):
    a, b = a.cpu().numpy(), b.cpu().numpy()
    assert np.all(np.isfinite(a))
    np.testing.assert_allclose(a, b, rtol=tol, atol=tol * max(1.0, np.abs(b).max()))


def _cloud(sg, n, seed, masses=False):
    pr = random_pair(n, n, seed)
    m = np.random.default_rng(seed).uniform(0.5, 2.0, n) if masses else None
    return sg.Cloud(pr.tmpl, m)


# template sizes around one block (1 024 points), where the points per thread
# change (16 384, 131 072) and the end of the loop's range
@pytest.mark.parametrize("M,g_mode,masses,E", [(40, 0, False, 3), (1024, 1, True, 8), (1025, 0, False, 1),
                                               (2049, 0, True, 9), (16384, 1, False, 5), (16385, 0, False, 5),
                                               (131073, 1, True, 4), (262144, 0, False, 3), (262145, 0, False, 3)])
def test_loop_matches_per_iteration_kernels(sg, both, M, g_mode, masses, E):
    tm, rf = _cloud(sg, M, 11 + M, masses), _cloud(sg, 600, 12, masses)
    prm = sg.Params(p=1.0, g_mode=g_mode, k=8, E=E, flags=SUMS, sigma=0.1, momentum=0.3 if M == 2049 else 0.0)
    (pa, sa), (pb, sb) = (c.register(tm, rf, prm, stats=True) for c in both)
    _close(pa, pb)
    _close(sa, sb)
    pc, _ = both[0].register(tm, rf, prm)              # without the energy sums: the same poses
    assert torch.equal(pa, pc)


def test_loop_from_a_given_pose_and_repeated(sg, both):
    """In place from a non-identity pose; a second call continues from it."""
    tm, rf = _cloud(sg, 5000, 1), _cloud(sg, 3000, 2)
    prm = sg.Params(p=1.0, k=8, E=6, flags=SUMS)
    c, s = np.cos(0.3), np.sin(0.3)
    R = np.array([[c, -s, 0], [s, c, 0], [0, 0, 1.0]])
    poses = []
    for ctx in both:
        pose = sg.pose_from_srt(1.1, R, [0.1, -0.2, 0.3])
        for _ in range(2):
            ctx.register(tm, rf, prm, pose=pose)
        poses.append(pose)
    _close(*poses)


def test_loop_batch_and_multistart(sg, both):
    sizes = [(60, 50), (1024, 900), (1300, 3000), (9000, 2000), (40, 700), (5000, 5000)]
    tms = [_cloud(sg, m, 100 + m) for m, _ in sizes]
    rfs = [_cloud(sg, n, 200 + n) for _, n in sizes]
    prm = sg.Params(p=1.0, k=8, E=7, flags=SUMS)
    res = [c.register_batch(tms, rfs, prm, stats=True) for c in both]
    for a, b in zip(*res):
        _close(a, b)
    # each member as by itself (the sums in other chunks: FP64 rounding)
    for r in range(len(sizes)):
        pose, _ = both[0].register(tms[r], rfs[r], prm)
        _close(res[0][0][r], pose)
    pr = config1(n=3000)
    tm, rf = sg.Cloud(pr.tmpl), sg.Cloud(pr.ref)
    R0 = super_fibonacci_rotations(5)
    a, b = (c.multistart(tm, rf, prm, R0) for c in both)
    _close(a[0], b[0])
    _close(a[1], b[1])
    assert a[2] == b[2]


def test_loop_pyramid_and_vector(sg, both):
    pr = config1(n=2500)
    tm, rf = sg.Cloud(pr.tmpl), sg.Cloud(pr.ref)
    levels = [sg.Level(0.5, 1.0, 3), sg.Level(0.0, 0.5, 4, 8), sg.Level(0.25, 0.5, 2)]
    prm = sg.Params(p=1.0, k=8, E=9, flags=SUMS)
    (pa, sa), (pb, sb) = (c.register_pyramid(tm, rf, prm, levels, stats=True) for c in both)
    _close(pa, pb)
    _close(sa, sb)
    hX, hY = (both[0].descriptors_hn(c, 16, 8) for c in (rf, tm))
    pa, pb = (c.register_vec(tm, hY, rf, hX, prm)[0] for c in both)
    _close(pa, pb)


def test_loop_degenerate_and_nonfinite_inputs_are_errors(sg, both):
    pr = config1(n=2000)
    flat = pr.tmpl.copy()
    flat[:] = flat[0]
    bad = pr.tmpl.copy()
    bad[7, 1] = np.nan
    prm = sg.Params(p=1.0, k=8, E=4, flags=SUMS)
    for ctx in both:
        for t in (flat, bad):
            with pytest.raises(sg.SgrError):
                ctx.register(sg.Cloud(t), sg.Cloud(pr.ref), prm)
        ctx.register(sg.Cloud(pr.tmpl), sg.Cloud(pr.ref), prm)   # usable afterwards
