"""Scratch that a call can do without, where it cannot be had."""
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


def test_unrolled_backward_in_a_capture_that_cannot_grow_the_scratch(sg):
    """A segment's forces are kept only where there is room: with scratch from a
    call of one-iteration segments the captured call evaluates them again, and
    gives the same bits."""
    ctx = sg.Context(0)
    rng = np.random.default_rng(5)
    n, E = 8192, 200
    u = rng.normal(size=(n, 3))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    tm, rf = sg.Cloud(u.astype(np.float32)), sg.Cloud((u * 1.05 + 0.02).astype(np.float32))
    (a_t, m_t), (a_r, m_r) = (ctx.descriptors(c, 16) for c in (tm, rf))
    ctx.close()
    ctx = sg.Context(0)                 # its scratch is that of the calls below
    prm = sg.Params(p=1.0, k=16, E=E, sigma=0.05)
    grad = torch.linspace(0.5, 1.5, 13, dtype=torch.float64, device="cuda")
    args = (tm, a_t, rf, a_r, m_t, m_r, prm)
    ckpt = [ctx.unrolled_fwd(*args, k, sg.pose_identity())[1] for k in (1, E)]
    ctx.unrolled_bwd(*args, 1, ckpt[0], grad)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = ctx.unrolled_bwd(*args, E, ckpt[1], grad)
    outs = []
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        outs.append([x.clone() for x in out])
    want = ctx.unrolled_bwd(*args, E, ckpt[1], grad)
    for o in outs:
        assert all(torch.equal(a, b) for a, b in zip(o, want))
    ctx.close()
