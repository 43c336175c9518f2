"""Registrations whose one-launch loop gives up (a poll limit of 1, read when a
context is made) start again from their initial pose: the same result as the
loop's, up to the rounding of float64 sums in another order (1e-10 leaves four
digits over it through these few iterations).  Every call has a context of its
own, so that every one of them stalls."""
import os

import numpy as np
import pytest
import torch

from synth import config1, super_fibonacci_rotations

pytestmark = pytest.mark.gpu

SUMS = 8


@pytest.fixture(scope="module")
def sg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_01061_amd as sg
    return sg


def _both(sg, call):
    """What call(context) gives with the loop and after a stall."""
    out = []
    for spins in (None, "1"):
        if spins:
            os.environ["SGR_LOOP_SPINS"] = spins
        try:
            ctx = sg.Context(0)
        finally:
            os.environ.pop("SGR_LOOP_SPINS", None)
        out.append(call(ctx).cpu().numpy())
        ctx.close()
    np.testing.assert_allclose(out[1], out[0], rtol=1e-10, atol=1e-10)
    return out[0]


def _start(sg):
    c, s = np.cos(0.2), np.sin(0.2)
    return sg.pose_from_srt(1.1, np.array([[c, -s, 0], [s, c, 0], [0, 0, 1.0]]), [0.1, -0.2, 0.3])


@pytest.mark.parametrize("flags", [0, SUMS])
@pytest.mark.parametrize("iters", [(1, 5), (5, 1), (1, 1, 4), (3, 4)])
def test_pyramid(sg, flags, iters):
    """Levels of one iteration run without the all-pairs loop."""
    pr = config1(n=1500)
    tm, rf = sg.Cloud(pr.tmpl), sg.Cloud(pr.ref)
    levels = [sg.Level(0.0, 2.0 / (1 + i), n, 8 + 4 * i) for i, n in enumerate(iters)]
    prm = sg.Params(p=1.0, k=8, E=sum(iters), flags=flags)
    got = _both(sg, lambda c: c.register_pyramid(tm, rf, prm, levels, pose=_start(sg))[0])
    assert np.abs(got - _start(sg).cpu().numpy()).max() > 1e-3


@pytest.mark.parametrize("kind", ["single", "sums", "batch", "multistart", "vector"])
def test_other_registrations(sg, kind):
    pr = config1(n=2500)
    tm, rf = sg.Cloud(pr.tmpl), sg.Cloud(pr.ref)
    prm = sg.Params(p=1.0, k=8, E=5, flags=0 if kind == "single" else SUMS)

    def call(c):
        if kind == "batch":
            return c.register_batch([tm, rf], [rf, tm], prm)[0]
        if kind == "multistart":
            return c.multistart(tm, rf, prm, super_fibonacci_rotations(4))[0]
        if kind == "vector":
            h = [c.descriptors_hn(x, 16, 8) for x in (tm, rf)]
            return c.register_vec(tm, h[0], rf, h[1], prm, pose=_start(sg))[0]
        return c.register(tm, rf, prm, pose=_start(sg))[0]
    _both(sg, call)
