"""The first calls with new inputs run their iterations directly, the fourth in
a row captures them, later ones replay: all give the same bits, also when two
inputs alternate and when the inputs change behind the same addresses."""
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


def _cloud(sg, n, seed):
    return sg.Cloud((np.random.default_rng(seed).normal(size=(n, 3)) * [1, .7, .5]).astype(np.float32))


@pytest.mark.parametrize("kind", ["single", "batch", "vector"])
def test_direct_captured_and_replayed_runs_agree(sg, kind):
    ctx = sg.Context(0)
    prm = sg.Params(p=1.0, k=8, E=6)
    pairs = [(_cloud(sg, 700 + 31 * i, i), _cloud(sg, 900 + 17 * i, 10 + i)) for i in range(2)]
    desc = [[torch.linspace(0, 1, 4 * c.n, device="cuda").reshape(c.n, 4).sin().contiguous() for c in p] for p in pairs]
    poses = [sg.pose_identity().repeat(2, 1) for _ in pairs]
    first = sg.pose_identity().repeat(2, 1)

    def run(i):
        t, r = pairs[i]
        poses[i].copy_(first)
        if kind == "batch":
            return ctx.register_batch([t, r], [r, t], prm, poses=poses[i])[0].clone()
        if kind == "vector":
            return ctx.register_vec(t, desc[i][0], r, desc[i][1], prm, pose=poses[i][0])[0].clone()
        return ctx.register(t, r, prm, pose=poses[i][0])[0].clone()

    def fresh(i):
        other = sg.Context(0)
        nonlocal ctx
        ctx, keep = other, ctx
        try:
            return run(i)
        finally:
            ctx = keep
            other.close()

    want = [fresh(0), fresh(1)]
    for i in (0, 0, 0, 0, 0, 1, 0, 1, 1, 1, 1, 1, 0, 0):
        assert torch.equal(run(i), want[i]), i
    pairs[0][0].soa.copy_(_cloud(sg, pairs[0][0].n, 99).soa)      # the same addresses, other points
    want[0] = fresh(0)
    for _ in range(6):
        assert torch.equal(run(0), want[0])
    ctx.close()
