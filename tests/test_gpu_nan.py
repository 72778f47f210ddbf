"""GPU checks of soft masks with voxels that are not finite, against the
oracle.  A NaN voxel is outside and leaves the vertices on its edges without a
position: no diameter takes them in, and the diameters and maximising pairs are
those of the other vertices (exact on both sides, so equal).  An infinite voxel
is inside (or outside) like any other, with its vertices at the other voxel."""
import sys

import numpy as np
import pytest

from oracle import oracle as O
from paper_2510_02894_amd import synth

pytestmark = pytest.mark.gpu

SP = (1.25, 0.7, 0.75)


def say(msg):
    print("[case] " + msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def S():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_02894_amd import shape3d

    shape3d.load()
    yield shape3d
    shape3d.set_small_path(True)


def masks():
    g = np.random.default_rng(1)
    m = synth.soft_roi((33, 38, 41), g, 3, 4.0, 11.0, 1.0)

    def put(a, where, v):
        a = a.copy()
        a[where] = v
        return a

    lattice = np.zeros(m.shape, bool)
    lattice[::5, ::7, ::3] = True
    noise = g.random((12, 19, 35)).astype(np.float32)
    return [("nan lattice", put(m, lattice, np.nan)), ("nan 20 percent", put(m, g.random(m.shape) < 0.2, np.nan)),
            ("nan below half", put(m, m <= 0.5, np.nan)),
            ("noise with nan", put(noise, g.random(noise.shape) < 0.5, np.nan)),
            ("inf inside", put(m, m > 0.9, np.inf)), ("-inf outside", put(m, m < 0.1, -np.inf)),
            ("noise with inf", put(noise, g.random(noise.shape) < 0.1, np.inf)),
            ("all nan", np.full((6, 6, 6), np.nan, np.float32)), ("all inf", np.full((6, 6, 6), np.inf, np.float32))]


@pytest.mark.parametrize("name,m", masks(), ids=[k for k, _ in masks()])
def test_masks_that_are_not_finite(S, name, m):
    import torch

    vol = torch.from_numpy(m).cuda()
    with np.errstate(all="ignore"):
        ref = O.shape3d(m, SP)
    has = (ref["pair_ids"] >= 0).all(axis=1)  # diameters that some pair has
    for small in (True, False):
        say("%s, small path %s" % (name, small))
        S.set_small_path(small)
        f, st, rc = S.features(vol, SP, stats=True)
        assert rc == ref["status"] and st["V"] == ref["V"] and st["T"] == ref["T"]
        np.testing.assert_array_equal(st["pair_ids"], ref["pair_ids"])
        np.testing.assert_array_equal(f[2:][has], ref["features"][2:][has])


@pytest.mark.parametrize("scale", [1e-90, 1e78, 1e80])
def test_adjoint_where_a_normal_leaves_the_range(S, scale):
    """The squares of the triangles' normals are 0 or infinite: no area term,
    as the oracle's division by that length gives."""
    import torch

    p = np.full((4, 5, 6), 0.2, np.float32)
    p[1:3, 1:4, 2:4] = 0.8
    sp = (scale, 2 * scale, scale)
    g = np.array([0.0, 1.0, 0.0, 0.0, 0.0, 0.0])
    say("adjoint, spacing %g" % scale)
    t = torch.from_numpy(p).cuda()
    _, saved = S.soft_forward(t, sp)
    got = S.soft_backward(t, saved, g).cpu().numpy()
    with np.errstate(all="ignore"):
        exp = O.soft_grad(p, sp, g)
    assert np.all(exp == 0.0)
    np.testing.assert_array_equal(got, exp)
