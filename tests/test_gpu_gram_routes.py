"""GPU checks of the Gram pipeline, which calls take with prune = 0, with the
FP32 kernel, and on a caller's workspace that does not hold the block lists (then
with its own pruning, for prune 1 and 2): every tiling of the split-f16 kernel on
a single ROI, a batch, recorded, and with small plane buckets; the pruned pair
tiles and plane buckets against the oracle; the small path up to its 2^22 voxels.
Diameters and maximising pairs are exact, so they must be equal."""
import sys

import numpy as np
import pytest

from oracle import oracle as O
from paper_2510_02894_amd import synth

pytestmark = pytest.mark.gpu

TILINGS = [(it, jc) for it in (4, 8) for jc in (64, 128, 256, 512, 1024)]


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
    shape3d.set_tuning(8, 1024, 0, 1, prune=1)


def union(shape, seed, n=4, lo=10.0, hi=40.0):
    c = min(shape) / 2.0
    return synth.ellipsoid_union(shape, synth.ellipsoid_params(synth.rng(9, seed), n, lo, hi, 0.5 * c, 1.3 * c)).astype(np.uint8)


@pytest.mark.parametrize("it,jc", TILINGS)
def test_every_split_tiling_single(S, it, jc):
    import torch

    m = union((50, 66, 71), 1, lo=8.0, hi=28.0)
    sp = (1.1, 0.8, 0.9)
    ref = O.shape3d(m, sp)
    say("every pair, tiling %d x %d" % (it, jc))
    S.set_tuning(it, jc, 0, 1, prune=0)
    f, st, rc = S.features(torch.from_numpy(m).cuda(), sp, stats=True)
    assert rc == 0 and st["V"] == ref["V"]
    np.testing.assert_array_equal(f[2:], ref["features"][2:])
    np.testing.assert_array_equal(st["pair_ids"], ref["pair_ids"])


def test_every_split_tiling_batched_and_graph(S):
    import torch

    buf, offs, shapes, sps = synth.batched_rois(40, 7, lmin=8.0, lmax=48.0)
    base = torch.from_numpy(buf).cuda()
    table = S.roi_table(offs, shapes, sps)
    ref = np.array([O.shape3d(buf[o:o + int(np.prod(s))].reshape(s), sp)["features"][2:]
                    for o, s, sp in zip(offs, shapes, sps)])
    for it, jc in TILINGS:
        for bpc in (0, 1):
            say("every pair, batch, tiling %d x %d, %d blocks/CU" % (it, jc, bpc))
            S.set_tuning(it, jc, bpc, 1, prune=0)
            for graph in (False, True, True):
                np.testing.assert_array_equal(S.batched(base, table, graph=graph)[0][:, 2:], ref)


def test_small_buckets_of_every_pair(S):
    """More than 2^16 plane buckets: those of few rows have a kernel of their own."""
    buf, offs, shapes, sps = synth.batched_rois_torch(400, 11, lmin=40.0, lmax=64.0)
    assert sum(2 * (d[0] + d[1] + d[2]) + 3 for d in shapes) >= 1 << 16
    table = S.roi_table(offs, shapes, sps)
    S.set_tuning(8, 1024, 0, 1, prune=1)
    ref, _, ref_st = S.batched(buf, table, stats=True)
    for it, jc, kern in [(8, 512, 1), (4, 64, 1), (8, 128, 0)]:
        say("every pair, 400 ROIs, tiling %d x %d kernel %d" % (it, jc, kern))
        S.set_tuning(it, jc, 0, kern, prune=0)
        out, status, st = S.batched(buf, table, stats=True)
        assert np.all(status == 0)
        np.testing.assert_array_equal(out, ref)
        for r in range(len(offs)):
            np.testing.assert_array_equal(st[r]["pair_ids"], ref_st[r]["pair_ids"], err_msg="ROI %d" % r)
    host = buf.cpu().numpy()
    for r in (3, 250):
        m = host[offs[r]:offs[r] + int(np.prod(shapes[r]))].reshape(shapes[r])
        np.testing.assert_array_equal(ref[r, 2:], O.shape3d(m, sps[r])["features"][2:])


# With dims of at most 4,000 a ROI may have a million bricks, whose vertices the
# block lists pad to 32 rows each: a workspace for 800,000 vertices a ROI then
# holds the vertex rows of the Gram pipeline and not the lists.
SIDE, ROOM = 4000, 800000


@pytest.mark.parametrize("prune", [1, 2])
@pytest.mark.parametrize("dtype", ["uint8", "float32"])
def test_pruned_on_a_workspace_without_room_for_the_lists(S, prune, dtype):
    import torch

    g = np.random.default_rng(17)
    if dtype == "uint8":
        c = np.indices((60, 61, 62)).astype(np.float64) - 30.0
        ms = [union((90, 110, 120), 3, lo=20.0, hi=50.0), ((c ** 2).sum(0) <= 27.0 ** 2).astype(np.uint8),
              synth.box_mask((32, 22, 27), (1, 1, 1), (30, 20, 25)), synth.random_mask((30, 31, 29), 0.3, g),
              synth.box_mask((3, 4, 5), (1, 1, 1), (1, 1, 1))]
        sps = [(1.25, 0.7, 0.75), (1.0, 1.0, 1.0), (1.0, 1.0, 1.0), (0.9, 1.0, 1.1), (1.0, 1.0, 1.0)]
    else:
        ms = [synth.soft_roi((70, 80, 75), g, 4, 10.0, 25.0, 1.0), synth.differentiable_small(3)[0].astype(np.float32)]
        sps = [(1.25, 0.7, 0.75), (1.0, 1.0, 1.0)]
    n = len(ms)
    base = torch.from_numpy(np.concatenate([m.ravel() for m in ms])).cuda()
    offs = np.concatenate([[0], np.cumsum([m.size for m in ms])[:-1]])
    tab = S.table_to_device(S.roi_table_ex(offs, [m.shape for m in ms], sps))
    S.set_prune(prune)
    md = (SIDE, SIDE, SIDE)
    dt = S.U8 if dtype == "uint8" else S.F32
    ws = torch.empty(S.batched_workspace_size(n, md, dt, n * ROOM), dtype=torch.uint8, device="cuda")
    say("pruned Gram pipeline, prune %d, %s: workspace of %.2f GB" % (prune, dtype, ws.numel() / 1e9))
    out, status = S.batched_dev(base, tab, n, md, workspace=ws)
    out = out.cpu().numpy()
    assert np.all(status.cpu().numpy() == 0)
    for r, (m, sp) in enumerate(zip(ms, sps)):
        np.testing.assert_array_equal(out[r], S.features(torch.from_numpy(m).cuda(), sp), err_msg="ROI %d" % r)
        if m.size < 300000:
            np.testing.assert_array_equal(out[r, 2:], O.shape3d(m, sp)["features"][2:], err_msg="ROI %d" % r)


@pytest.mark.parametrize("kernel,prune", [(1, 0), (0, 1)])
@pytest.mark.parametrize("shape", [(41, 40, 41), (64, 64, 64), (45, 301, 70), (161, 161, 161)], ids=str)
def test_small_path_beside_every_pair(S, shape, kernel, prune):
    """Up to 2^22 voxels and 16,384 vertices where the other way visits every pair."""
    import torch

    c = np.indices(shape).astype(np.float64)
    m = (sum(((c[k] - shape[k] / 2.0) / (0.28 * min(shape) + 2.0 * k)) ** 2 for k in range(3)) <= 1.0).astype(np.uint8)
    m[0, 0, 0] = m[-1, -1, -1] = 1
    vol = torch.from_numpy(m).cuda()
    sp = (1.0, 0.8, 1.2)
    S.set_tuning(8, 1024, 0, kernel, prune=prune)
    got = []
    for small in (False, True):
        say("%s, kernel %d, prune %d, small path %s" % (shape, kernel, prune, small))
        S.set_small_path(small)
        f, st, rc = S.features(vol, sp, stats=True)
        got.append((f.tolist(), st["pair_ids"].tolist(), st["V"], st["T"], st["pairs_2d"], rc))
    assert got[0] == got[1]
    if m.size < 1000000:
        ref = O.shape3d(m, sp)
        np.testing.assert_array_equal(got[1][0][2:], ref["features"][2:])
        np.testing.assert_array_equal(got[1][1], ref["pair_ids"])
