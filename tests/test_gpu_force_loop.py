"""The small all-pairs registration, all iterations in one launch, against the
per-iteration kernels (a context whose loop gives up at once runs those): the
FP32 pair sums have the same bits, FP64 sums another order."""
import os

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


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


def _surface(n, seed):
    rng = np.random.default_rng(seed)
    u = rng.normal(size=(n, 3))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    return (u * [1.0, 0.7, 0.4] + rng.normal(size=(n, 3)) * 0.02).astype(np.float32)


def _close(a, b):
    a, b = a.cpu().numpy(), b.cpu().numpy()
    assert np.all(np.isfinite(a))
    np.testing.assert_allclose(a, b, rtol=1e-10, atol=1e-10)


@pytest.mark.parametrize("m,n", [(9, 9), (100, 2000), (255, 257), (256, 16), (257, 1000), (1024, 1024), (1025, 1023),
                                 (2048, 2048), (2048, 4099), (700, 20001), (300, 9)])
@pytest.mark.parametrize("g_mode,masses", [(0, False), (1, True), (2, True)])
def test_loop_equals_the_steps(sg, both, m, n, g_mode, masses):
    """Three iterations: a difference of FP64 rounding grows by far less than
    1e5 in so few."""
    rng = np.random.default_rng(m)
    w = [rng.uniform(0.5, 2.0, c) if masses else None for c in (m, n)]
    t, r = sg.Cloud(_surface(m, 1), masses=w[0]), sg.Cloud(_surface(n, 2), masses=w[1])
    prm = sg.Params(p=1.0, g_mode=g_mode, k=8, E=3, momentum=0.3)
    a, b = (c.register(t, r, prm)[0] for c in both)
    _close(a, b)


@pytest.mark.parametrize("sigma", [1e-3, 3e-4])
def test_loop_with_curvatures_far_apart(sg, both, sigma):
    """A sigma far below the curvatures' spread: blocks whose exponent cannot
    be expanded, weights that underflow."""
    t, r = sg.Cloud(_surface(900, 3)), sg.Cloud(_surface(1100, 4))
    prm = sg.Params(p=1.0, k=8, E=4, sigma=sigma)
    a, b = (c.register(t, r, prm)[0] for c in both)
    _close(a, b)


def test_loop_in_a_pyramid_and_repeated(sg, both):
    t, r = sg.Cloud(_surface(800, 5)), sg.Cloud(_surface(1200, 6))
    prm = sg.Params(p=1.0, k=8, E=9)
    levels = [sg.Level(radius_scale=0.0, sigma_scale=2.0, iters=4, k=16),
              sg.Level(radius_scale=0.0, sigma_scale=1.0, iters=5, k=8)]
    out = []
    for c in both:
        out.append([c.register_pyramid(t, r, prm, levels)[0] for _ in range(3)])
    for a, b in zip(*out):
        _close(a, b)
        assert torch.equal(a, out[0][0])

