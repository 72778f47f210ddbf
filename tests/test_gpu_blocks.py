"""GPU checks of the block-pair pass (the default route of every call but the
small single ROIs): equal to the pass over every pair, and to the oracle, at
the sizes where its blocks, superblocks and list can go wrong (one block, a
block's and a superblock's edge, a list that is too short), for strided crops,
labels and soft masks, and for spacings far from 1.  Diameters and maximising
pairs are exact on both sides, so they must be equal."""
import sys

import numpy as np
import pytest

from oracle import oracle as O
from paper_2510_02894_amd import synth

pytestmark = pytest.mark.gpu


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
    shape3d.set_small_path(False)
    yield shape3d
    shape3d.set_small_path(True)
    shape3d.set_prune(1)


def ball(n, r):
    c = (n - 1) / 2.0
    z, y, x = np.mgrid[:n, :n, :n]
    return (((z - c) ** 2 + (y - c) ** 2 + (x - c) ** 2) <= r * r).astype(np.uint8)


def rod(n):
    """A rod of n voxels: 4 n + 2 vertices."""
    m = np.zeros((1, 1, n), np.uint8)
    m[0, 0, :] = 1
    return m


def shapes():
    g = np.random.default_rng(23)
    out = [("rod %d" % n, rod(n), (1.0, 0.7, 1.3)) for n in (1, 7, 8, 127, 128, 135)]
    out += [("plate", np.ones((1, 40, 37), np.uint8), (2.0, 1.0, 0.9)),
            ("random 9x70x33", synth.random_mask((9, 70, 33), 0.4, g), (1.0, 1.1, 0.6)),
            ("ball r=18", ball(40, 18), (1.0, 1.0, 1.0)),
            ("union", synth.ellipsoid_union((50, 70, 65), synth.ellipsoid_params(g, 3, 6.0, 24.0, 12.0, 45.0)).astype(np.uint8),
             (1.1, 0.8, 0.9)),
            ("soft", synth.soft_roi((33, 38, 41), g, 3, 4.0, 11.0, 1.0), (1.25, 0.7, 0.75)),
            ("soft noise", g.random((12, 19, 35)).astype(np.float32), (1.0, 1.2, 0.9))]
    return out


@pytest.mark.parametrize("name,m,sp", shapes(), ids=[s[0] for s in shapes()])
def test_equals_every_pair_and_oracle(S, name, m, sp):
    import torch

    vol = torch.from_numpy(m).cuda()
    say("blocks: " + name)
    S.set_prune(0)
    f0, st0, rc0 = S.features(vol, sp, stats=True)
    S.set_prune(1)
    f1, st1, rc1 = S.features(vol, sp, stats=True)
    assert rc0 == rc1
    np.testing.assert_array_equal(f1, f0)
    np.testing.assert_array_equal(S.features(vol, sp), f1)  # without statistics
    np.testing.assert_array_equal(st1["pair_ids"], st0["pair_ids"])
    assert (st1["V"], st1["T"], st1["pairs_2d"]) == (st0["V"], st0["T"], st0["pairs_2d"])
    ref = O.shape3d(m, sp)
    np.testing.assert_array_equal(f1[2:], ref["features"][2:])
    np.testing.assert_array_equal(st1["pair_ids"], ref["pair_ids"])


def test_block_list_too_short(S):
    """A ball, whose blocks all have far partners: more block pairs than the
    list holds (they are evaluated where they are found, and the ties taken in
    a second enumeration)."""
    import torch

    m = ball(158, 77)
    vol = torch.from_numpy(m).cuda()
    say("blocks: ball r=77")
    S.set_prune(0)
    f0, st0, _ = S.features(vol, (1.0, 1.0, 1.0), stats=True)
    S.set_prune(1)
    f1, st1, _ = S.features(vol, (1.0, 1.0, 1.0), stats=True)
    np.testing.assert_array_equal(f1, f0)
    np.testing.assert_array_equal(st1["pair_ids"], st0["pair_ids"])


@pytest.mark.parametrize("sp", [(1e-25, 2e-25, 1e-25), (3e20, 1e20, 2e20), (1.0, 1e-12, 1e-12), (1e-3, 1e6, 1.0)])
def test_spacings_far_from_one(S, sp):
    import torch

    m = ball(30, 12)
    S.set_prune(1)
    say("blocks: spacing %s" % (sp,))
    f, st, _ = S.features(torch.from_numpy(m).cuda(), sp, stats=True)
    ref = O.shape3d(m, sp)
    np.testing.assert_array_equal(f[2:], ref["features"][2:])
    np.testing.assert_array_equal(st["pair_ids"], ref["pair_ids"])


@pytest.mark.parametrize("workspace", [False, True])
def test_crops_and_labels(S, workspace):
    import torch

    lab = synth.label_map(4, (30, 41, 50), 5, 3.0, 12.0, noise=0.001)
    dev = torch.from_numpy(lab).cuda()
    sp = (1.0, 0.8, 1.2)
    lo, hi = (3, 5, 7), (28, 39, 46)
    shape = [h - l for l, h in zip(lo, hi)]
    off = (lo[0] * 41 + lo[1]) * 50 + lo[2]
    n = 6  # labels 1..5, then every nonzero voxel
    labels = [1, 2, 3, 4, 5, 0]
    tab = S.roi_table_ex([off] * n, [shape] * n, [sp] * n, strides=[(41 * 50, 50)] * n, labels=labels)
    ws = None
    if workspace:
        ws = torch.empty(S.batched_workspace_size(n, shape, S.U8, 60000), dtype=torch.uint8, device="cuda")
    S.set_prune(1)
    say("blocks: crops, workspace %s" % workspace)
    out, status = S.batched_dev(dev.view(-1), S.table_to_device(tab), n, shape, workspace=ws)
    out, status = out.cpu().numpy(), status.cpu().numpy()
    crop = lab[lo[0]:hi[0], lo[1]:hi[1], lo[2]:hi[2]]
    for r, l in enumerate(labels):
        m = (crop == l if l else crop != 0).astype(np.uint8)
        ref = O.shape3d(m, sp)
        assert status[r] == ref["status"]
        np.testing.assert_array_equal(out[r, 2:], ref["features"][2:], err_msg="label %d" % l)
