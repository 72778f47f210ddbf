"""GPU checks of the longest rows a volume may have (32,767 voxels along axis 2:
1,024 row-groups of 32 cubes, whose tile words are most of a mesh-pass
workgroup's LDS), forward and backward, against the oracle."""
import sys

import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu

SP = (1.1, 0.8, 0.95)


def say(msg):
    print("[case] " + msg, flush=True)
    sys.stdout.flush()


@pytest.fixture()
def S():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_02894_amd import shape3d

    shape3d.load()
    shape3d.set_small_path(False)
    yield shape3d
    shape3d.set_small_path(True)
    shape3d.set_prune(1)


def mask(shape, seed):
    g = np.random.default_rng(seed)
    p = np.where(g.random(shape) < 0.015, 0.6 + 0.4 * g.random(shape), 0.4 * g.random(shape)).astype(np.float32)
    p[0, 0, 0] = p[-1, -1, -1] = 0.9
    return p


@pytest.mark.parametrize("shape", [(2, 2, 32767), (9, 2, 32766)], ids=str)
@pytest.mark.parametrize("soft", [False, True])
def test_longest_rows(S, shape, soft):
    import torch

    p = mask(shape if not soft or shape[0] == 2 else (3, 2, 32766), 5)
    m = p if soft else (p > 0.5).astype(np.uint8)
    vol = torch.from_numpy(m).cuda()
    ref = O.shape3d(m, SP)
    for prune in (1, 0):
        say("long rows %s, soft %s, prune %d" % (m.shape, soft, prune))
        S.set_prune(prune)
        f, st, rc = S.features(vol, SP, stats=True)
        assert (rc, st["V"], st["T"]) == (ref["status"], ref["V"], ref["T"])
        np.testing.assert_allclose(f[:2], ref["features"][:2], rtol=1e-9)
        np.testing.assert_array_equal(f[2:], ref["features"][2:])
        np.testing.assert_array_equal(st["pair_ids"], ref["pair_ids"])
    if soft:
        S.set_prune(1)
        w = np.array([0.7, -0.3, 0.9, 0.4, -0.5, 0.6])
        _, saved = S.soft_forward(vol, SP)
        got = S.soft_backward(vol, saved, w).cpu().numpy()
        exp = O.soft_grad(m, SP, w)
        assert np.abs(got - exp).max() <= 2e-6 * np.abs(exp).max()
    else:
        # axis lengths to 1e-6 of the longest, their ratios to 1e-6 (two eigensolvers)
        got, exp = S.shape_class(vol, SP), O.shape_class(m, SP)["features"]
        np.testing.assert_allclose(got[:12], exp[:12], rtol=1e-9)
        np.testing.assert_allclose(got[12:15], exp[12:15], rtol=1e-9, atol=1e-6 * exp[12])
        np.testing.assert_allclose(got[15:], exp[15:], rtol=1e-9, atol=1e-6)
