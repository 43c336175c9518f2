"""The adjoint's fused launches at the edges of their blocks, and the unrolled
registration with and without its segments' forces kept."""
import numpy as np
import pytest
import torch

from oracle import ref as O

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
    return torch.as_tensor(np.asarray(x)).to(device="cuda", dtype=dtype).contiguous()


def _mom(P):
    c, S, lam = O.moments(P)
    return np.array([c[0], c[1], c[2], S[0, 0], S[1, 1], S[2, 2], S[0, 1], S[0, 2], S[1, 2], lam])


@pytest.mark.parametrize("m", [3, 255, 256, 257, 1023, 1025, 2049])
@pytest.mark.parametrize("n", [5, 257, 5000])
@pytest.mark.parametrize("p", [1.0, 2.0])
def test_force_adjoint_at_block_edges(sg, ctx, m, n, p):
    """Against the oracle's FP64 adjoint, 1e-4 in norm: FP32 pair terms carry
    about 1e-7 each, and the sums here cancel by less than a thousand."""
    rng = np.random.default_rng(m * 7 + n)
    Y, X = (rng.normal(size=(c, 3)).astype(np.float32) for c in (m, n))
    aY, aX = (rng.uniform(0.01, 0.3, c).astype(np.float32) for c in (m, n))
    wY, wX = (rng.uniform(0.5, 2.0, c).astype(np.float32).astype(np.float64) for c in (m, n))
    gf = rng.normal(size=(m, 3)).astype(np.float32)
    gF, gK = rng.normal(size=3), rng.normal(size=(3, 3))
    G = 2500.0
    prm = sg.Params(p=p, sigma=0.1, eps=0.05)
    tm, rf = sg.Cloud(Y, masses=wY), sg.Cloud(X, masses=wX)
    mom = _dev(_mom(X), torch.float64)
    f, w = ctx.force_fwd(tm, _dev(aY), rf, _dev(aX), mom, prm, G)
    gy, gm, gse = ctx.force_bwd(tm, _dev(aY), rf, _dev(aX), mom, prm, G, f, _dev(gf),
                                _dev(np.concatenate([gF, gK.reshape(-1)]), torch.float64))
    S = O.make_setup(X, Y, O.Params(p=p, sigma=0.1, eps=0.05), aX=aX.astype(np.float64), aY=aY.astype(np.float64),
                     wX=wX, mY=wY)
    want = O.force_vjp(Y.astype(np.float64), S, G, gf.astype(np.float64), gF, gK)
    for got, ref in zip((gy, gm), want):
        assert np.linalg.norm(got.cpu().numpy() - ref) <= 1e-4 * np.linalg.norm(ref)
    assert gse[0].item() == pytest.approx(want[2], rel=1e-4, abs=1e-4 * abs(want[2]))


def test_unrolled_with_and_without_kept_forces(sg, ctx):
    """8 000 000 template points: the forces of three iterations (288 MB) are
    evaluated again, those of two or one are kept; the checkpoints' spacing
    changes nothing else, so the gradients have the same bits."""
    rng = np.random.default_rng(4)
    m, n, E = 8_000_000, 64, 3
    Y = torch.from_numpy(rng.normal(size=(n, 3)).astype(np.float32)).cuda()
    Y = (Y.repeat(m // n, 1) + 0.1 * torch.sin(torch.arange(3 * m, device="cuda").reshape(m, 3) * 0.37)).contiguous()
    tm, rf = sg.Cloud(Y), sg.Cloud(rng.normal(size=(n, 3)).astype(np.float32))
    ay, ax = torch.rand(m, device="cuda") * 0.2, _dev(rng.uniform(0, 0.2, n))
    my, mx = (_dev(np.r_[0.0, 0.0, 0.0, 1.0, 0.9, 0.8, 0.0, 0.0, 0.0, 1.0], torch.float64) for _ in range(2))
    prm = sg.Params(p=2.0, sigma=0.1, eps=0.1, E=E)
    out = []
    for K in (3, 2, 1):
        pose, ckpt = ctx.unrolled_fwd(tm, ay, rf, ax, my, mx, prm, K)
        gp, gse = ctx.unrolled_bwd(tm, ay, rf, ax, my, mx, prm, K, ckpt, torch.linspace(-1, 1, 13))
        assert torch.isfinite(gp).all() and torch.isfinite(gse).all()
        out.append((pose, gp, gse))
    for o in out[1:]:
        assert all(torch.equal(a, b) for a, b in zip(o, out[0]))
