"""The statistics a registration starts from, at the sizes where their kernels
change: 16 waves as one block or as 16 blocks (above 16 384 points), loads in
flight past the end of a cloud, four descriptor components read at once or one
by one, and the list of far descriptor rows in words of 64 rows."""
import numpy as np
import pytest
import torch

from oracle import ref as O
from parity_bars import F_TOL

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


def _dev(x, dtype=torch.float32):
    return torch.as_tensor(np.ascontiguousarray(x)).to(device="cuda", dtype=dtype)


@pytest.mark.parametrize("n", [4, 1023, 1025, 8191, 8193, 16384, 16385, 20481, 150001])
def test_moments(sg, ctx, n):
    """1e-12 of the largest coordinate: a thread adds at most 150 terms."""
    P = (np.random.default_rng(n).normal(size=(n, 3)) * [3.0, 2.0, 1.0] + [5.0, -1.0, 0.5]).astype(np.float32)
    _, mom = ctx.descriptors(sg.Cloud(P), 4)
    mom = mom.cpu().numpy()
    x = P.astype(np.float64)
    C = np.cov(x.T, bias=True)
    want = np.concatenate([x.mean(0), C[[0, 1, 2, 0, 0, 1], [0, 1, 2, 1, 2, 2]], [np.linalg.eigvalsh(C)[-1]]])
    np.testing.assert_allclose(mom, want, rtol=1e-12, atol=1e-12 * 20)


@pytest.mark.parametrize("m,n,g_mode,masses", [(300, 16385, 0, False), (300, 16385, 1, False), (300, 16385, 1, True),
                                               (300, 16384, 0, False), (300, 16385, 2, True), (16385, 300, 0, True)])
def test_first_iteration_of_a_large_registration(sg, ctx, m, n, g_mode, masses):
    """One iteration from clouds half a unit apart against the oracle's, which
    has the same curvatures: FP32 forces are within F_TOL of their scale, and
    here the scale is within ten times the net force that moves the points."""
    rng = np.random.default_rng(3)
    Y, X = ((rng.normal(size=(c, 3)) * [1, .7, .5]).astype(np.float32) for c in (m, n))
    Y[:, 0] += np.float32(0.5)
    my, mx = (rng.uniform(0.5, 2.0, c) if masses else None for c in (m, n))
    my, mx = (None if w is None else w.astype(np.float32).astype(np.float64) for w in (my, mx))
    ty, tx = sg.Cloud(Y, masses=my), sg.Cloud(X, masses=mx)
    a_y, _ = ctx.descriptors(ty, 6)
    a_x, _ = ctx.descriptors(tx, 6)
    got, _ = ctx.register(ty, tx, sg.Params(p=1.0, g_mode=g_mode, k=6, E=1))
    S = O.make_setup(X, Y, O.Params(p=1.0, g_mode=g_mode, k=6, E=1), aX=a_x.cpu().numpy().astype(np.float64),
                     aY=a_y.cpu().numpy().astype(np.float64), wX=mx, mY=my)
    Y64 = Y.astype(np.float64)
    want = O.compose(O.Pose(1.0, np.eye(3), np.zeros(3)), O.step(Y64, S, 0), Y64.mean(axis=0)).apply(Y)
    g = got.cpu().numpy()
    moved = O.Pose(g[0], g[1:10].reshape(3, 3), g[10:13]).apply(Y)
    assert np.linalg.norm(moved - want) <= 10 * F_TOL * np.linalg.norm(want - Y64)


@pytest.mark.parametrize("n", [5, 1024, 1100, 5000])
@pytest.mark.parametrize("D", [4, 8, 16, 28])
def test_descriptor_rows_at_any_alignment(sg, ctx, n, D):
    """Rows on a 16-byte boundary are read four components at a time, others
    one by one; the additions are the same."""
    rng = np.random.default_rng(D)
    Y, X = (rng.normal(size=(c, 3)).astype(np.float32) for c in (2 * n, n))
    ty, tx = sg.Cloud(Y), sg.Cloud(X)
    _, my = ctx.descriptors(ty, 4)
    _, mx = ctx.descriptors(tx, 4)
    ay, ax = _dev(rng.normal(size=(2 * n, D))), _dev(rng.normal(size=(n, D)))
    off = torch.empty(n * D + 1, device="cuda")
    off[1:] = ax.reshape(-1)
    ax_off = off[1:].view(n, D)
    assert ax_off.data_ptr() % 16 == 4
    prm = sg.Params(p=1.0, k=4, E=10, sigma=0.0)
    one = ctx.step_vec(ty, ay, tx, ax, my, mx, prm, 3, sg.pose_identity(), want_wrench=True)
    two = ctx.step_vec(ty, ay, tx, ax_off, my, mx, prm, 3, sg.pose_identity(), want_wrench=True)
    assert torch.isfinite(one[1]).all()
    assert torch.equal(one[0], two[0]) and torch.equal(one[1], two[1])


@pytest.mark.parametrize("m", [1, 64, 65, 65536, 70001])
def test_far_rows_in_any_word(sg, ctx, m):
    """All reference rows and half of the template's lie 25 spreads from the
    mean, the template's with reference partners: a row left out of the list
    would have no force.  The rows of the whole template against the same rows
    in two shorter ones (FP32 forces: 2e-5)."""
    rng = np.random.default_rng(m)
    n, D = 64, 4
    Y, X = (rng.normal(size=(c, 3)).astype(np.float32) for c in (m, n))
    ax = np.where(np.arange(n)[:, None] % 2, 0.5, 0.0) + rng.normal(size=(n, D)) * 1e-3
    side = rng.integers(0, 4, m)
    side[-1] = 1
    ay = np.select([side == 0, side == 1], [0.0, 0.5], 0.25)[:, None] + rng.normal(size=(m, D)) * 1e-3
    tx = sg.Cloud(X)
    _, mx = ctx.descriptors(tx, 4)
    my = _dev(np.r_[np.zeros(3), np.ones(3), np.zeros(3), 1.0], torch.float64)
    prm = sg.Params(p=1.0, k=4, E=10, sigma=0.01)

    def force(lo, hi):
        return ctx.step_vec(sg.Cloud(Y[lo:hi]), _dev(ay[lo:hi]), tx, _dev(ax), my, mx, prm, 3, sg.pose_identity(),
                            want_f=True)[2].cpu().numpy()
    f = force(0, m)
    assert (np.abs(f[side < 2]).max(1) > 0).all()
    if m > 1:
        h = m // 2 + 7
        np.testing.assert_allclose(f, np.concatenate([force(0, h), force(h, m)]), rtol=2e-5,
                                   atol=2e-5 * np.abs(f).max())


@pytest.mark.parametrize("n,k", [(9, 9), (63, 8), (64, 24), (65, 7), (129, 17)])
def test_normal_histograms_at_block_edges(sg, ctx, n, k):
    """FP32 rounding of the oracle's FP64 histograms: 3e-8 for weights up to
    one, where the normals are determined."""
    rng = np.random.default_rng(n)
    P = np.stack([rng.uniform(-1, 1, n), rng.uniform(-1, 1, n), 0.05 * rng.normal(size=n)], 1).astype(np.float32)
    h = ctx.descriptors_hn(sg.Cloud(P), k, 5).cpu().numpy()
    np.testing.assert_allclose(h, O.normal_histograms(P, k, 5)[0], rtol=0, atol=6e-8)
