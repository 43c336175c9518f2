"""Neighbour lists, nearest points and residuals of clouds whose grid has nearly
all of its cells along one axis, or could: a stray point on each of the six
sides, a pipe, a strip and a thin long slab along each axis, exactly as brute
force gives them (FP32 keys, ties by index).  Also clouds so
small that the squares of their cells underflow."""
import numpy as np
import pytest
import torch

from oracle import ref as O
from test_gpu_grid import _nearest, _surface

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_01061_amd as sg
    return sg


@pytest.fixture(scope="module")
def ctx(sg):
    c = sg.Context(0)
    yield c
    c.close()


def _cloud(kind, axis, side, n):
    rng = np.random.default_rng(2)
    if kind == "stray point":
        P = _surface(n, 1)
        P[17] = 0
        P[17, axis] = side * 500
        return P
    if kind == "pipe":                 # 1 000 long, radius 0.5
        f = rng.uniform(0, 2 * np.pi, n)
        P = np.stack([rng.uniform(0, 1000, n), 0.5 * np.cos(f), 0.5 * np.sin(f)], 1)
    elif kind == "slab":               # 8 x 0.008 x 250, normal: dense in the middle
        P = rng.normal(size=(n, 3)) * [30, 1, 1e-3]
    else:                              # a strip 300 x 1
        P = np.stack([rng.uniform(0, 300, n), rng.uniform(0, 1, n), rng.normal(size=n) * 1e-3], 1)
    return np.roll(P, axis, axis=1).astype(np.float32)


LONG = [("stray point", a, s) for a in range(3) for s in (1, -1)] + [(k, a, 1) for k in ("pipe", "strip", "slab") for a in range(3)]


@pytest.mark.parametrize("kind,axis,side", LONG)
@pytest.mark.parametrize("n", [6000, 20000])      # a grid built by one block, and by many
def test_lists(sg, ctx, kind, axis, side, n):
    P, k = _cloud(kind, axis, side, n), 16
    q = np.unique(np.r_[np.arange(0, n, n // 400), 17])
    assert np.array_equal(ctx.knn(sg.Cloud(P), k).cpu().numpy()[q], O.knn_c(P, k, q))
    _, idx = ctx.descriptors_batch([sg.Cloud(P)], k, want_idx=True)
    assert np.array_equal(idx[0].cpu().numpy()[q], O.knn_c(P, k, q))


@pytest.mark.parametrize("kind,axis,side", LONG)
@pytest.mark.parametrize("n", [6000, 20000])
def test_nearest_points_and_residual(sg, ctx, kind, axis, side, n):
    """The residual is the FP64 mean over the points that brute force picks:
    1e-12 for sums of 700 squares of identically posed points."""
    X = _cloud(kind, axis, side, n)
    rng = np.random.default_rng(3)
    near = X[::n // 500]
    Y = np.concatenate([near + rng.normal(size=near.shape) * 0.01, near[::5] * 1.02,
                        rng.normal(size=(100, 3)) * 400]).astype(np.float32)
    zero = torch.zeros(len(Y), device="cuda"), torch.zeros(n, device="cuda")
    want, keys = _nearest(Y, X)
    for tau in (0.05, 1e18):
        _, nn, key = ctx.change_detect(sg.Cloud(Y), zero[0], sg.Cloud(X), zero[1], sg.pose_identity(), tau)
        hit = keys <= np.float32(tau * tau)
        assert np.array_equal(nn.cpu().numpy(), np.where(hit, want, -1))
        assert np.array_equal(key.cpu().numpy()[hit], keys[hit])
    nn, _ = _nearest(Y, X, fused=True)
    rmse = np.sqrt(((Y.astype(np.float64) - X[nn].astype(np.float64)) ** 2).sum(1).mean())
    assert ctx.residual(sg.Cloud(Y), sg.Cloud(X), sg.pose_identity()).item() == pytest.approx(rmse, rel=1e-12)


@pytest.mark.parametrize("scale", [1e-38, 1e-24, 1e-22, 1e-20, 1e-17])
@pytest.mark.parametrize("n", [3000, 20000])
def test_lists_of_clouds_whose_squares_underflow(sg, ctx, scale, n):
    """Cell sides whose FP32 square underflows; many keys are 0 (ties by index)."""
    P, k = np.concatenate([_surface(n, 5), np.float32([[3, 0, 0], [0, 30, 0]])]) * np.float32(scale), 16
    q = np.r_[np.arange(0, n, n // 300), n, n + 1]
    assert np.array_equal(ctx.knn(sg.Cloud(P), k).cpu().numpy()[q], O.knn_c(P, k, q))


@pytest.mark.parametrize("e", [16, 18.6, 18.9])
def test_nearest_points_of_queries_far_away(sg, ctx, e):
    """So many cells away that the square of the distance in cells overflows."""
    X = _surface(3000, 5)
    u = np.random.default_rng(7).normal(size=(100, 3))
    Y = (u / np.linalg.norm(u, axis=1, keepdims=True) * 10.0 ** e).astype(np.float32)
    _, nn, _ = ctx.change_detect(sg.Cloud(Y), torch.zeros(100, device="cuda"), sg.Cloud(X),
                                 torch.zeros(3000, device="cuda"), sg.pose_identity(), 1.5e19)
    assert np.array_equal(nn.cpu().numpy(), _nearest(Y, X)[0])


@pytest.mark.parametrize("crowd", [1, 8, 31, 32, 33, 63, 64, 65, 97, 1500])
def test_nearest_points_in_a_crowded_cell(sg, ctx, crowd):
    """Cells around the number of points from which a row of them is read as a
    whole, exact ties among them."""
    rng = np.random.default_rng(crowd)
    X = np.concatenate([np.round(rng.normal(size=(crowd, 3)) * 3) * 1e-3, [[100, 0, 0], [0, -80, 0], [0, 0, 60]],
                        rng.normal(size=(crowd // 2, 3)) * 1e-3 + [0, 0, 60]])
    X = X[rng.permutation(len(X))].astype(np.float32)
    Y = np.concatenate([X, np.round(rng.normal(size=(200, 3)) * 8) * 5e-4, rng.normal(size=(50, 3)) * 50,
                        rng.normal(size=(50, 3)) * 1e-3 + [0, 0, 60]]).astype(np.float32)
    want, keys = _nearest(Y, X)
    for tau in (0.002, 1e18):
        _, nn, _ = ctx.change_detect(sg.Cloud(Y), torch.zeros(len(Y), device="cuda"), sg.Cloud(X),
                                     torch.zeros(len(X), device="cuda"), sg.pose_identity(), tau)
        assert np.array_equal(nn.cpu().numpy(), np.where(keys <= np.float32(tau * tau), want, -1))
