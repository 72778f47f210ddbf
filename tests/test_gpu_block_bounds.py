"""GPU checks of the block-pair pass on round shapes, where every point of the
surface has a far partner: the bound from the distances to the ROI's centre
(against every pair and the oracle: centred and not, any spacing, soft, with NaN
voxels, single and batched, on a caller's workspace), that it keeps the list of
block pairs short, and the kernels that serve a list that is too short all the
same (device results), with packed and with 64-bit vertex ids.  Diameters and
maximising pairs are exact on both sides, so they must be equal."""
import sys

import numpy as np
import pytest

from oracle import oracle as O

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


def dist(shape, centre, scale=(1.0, 1.0, 1.0)):
    g = np.indices(shape).astype(np.float64)
    return np.sqrt(sum(((g[k] - centre[k]) * scale[k]) ** 2 for k in range(3)))


def shapes():
    b = dist((40, 41, 42), (19.5, 20.0, 20.5))
    off = dist((70, 45, 52), (20.0, 22.3, 30.9))
    s = (1.0 / (1.0 + np.exp((b - 17.0) / 1.0))).astype(np.float32)
    nan = s.copy()
    nan[::4, ::5, ::3] = np.nan
    two = np.minimum(dist((30, 30, 90), (14.0, 15.0, 13.0)), dist((30, 30, 90), (14.0, 15.0, 76.0)))
    half = (off <= 18.7) & (np.indices(off.shape)[1] < 22)
    return [("ball", (b <= 18.0).astype(np.uint8), (1.0, 1.0, 1.0)),
            ("ball off the centre", (off <= 18.7).astype(np.uint8), (1.0, 1.0, 1.0)),
            ("ball, round in mm", (dist((27, 45, 41), (13.0, 22.0, 20.0), (1.5, 0.8, 0.9)) <= 17.0).astype(np.uint8), (1.5, 0.8, 0.9)),
            ("ball, small spacings", (b <= 18.0).astype(np.uint8), (1e-12, 1.0, 1e-3)),
            ("shell", ((b <= 18.0) & (b >= 16.5)).astype(np.uint8), (1.0, 1.0, 1.0)),
            ("half ball", half.astype(np.uint8), (1.0, 1.0, 1.0)),
            ("two balls", (two <= 12.0).astype(np.uint8), (1.0, 1.0, 1.0)),
            ("cylinder", np.repeat((b[20] <= 17.0)[None], 35, 0).astype(np.uint8), (1.0, 1.0, 1.0)),
            ("soft ball", s, (1.0, 1.0, 1.0)), ("soft ball, spacing", s, (1.25, 0.7, 0.75)),
            ("soft ball with nan", nan, (1.0, 1.0, 1.0))]


def reference(m, sp):
    with np.errstate(all="ignore"):
        return O.shape3d(m, sp)


@pytest.mark.parametrize("name,m,sp", shapes(), ids=[s[0] for s in shapes()])
def test_round_shapes(S, name, m, sp):
    import torch

    vol = torch.from_numpy(m).cuda()
    say("bounds: " + name)
    ref = reference(m, sp)
    S.set_prune(1)
    f, st, rc = S.features(vol, sp, stats=True)
    assert rc == ref["status"]
    np.testing.assert_array_equal(f[2:], ref["features"][2:])
    np.testing.assert_array_equal(st["pair_ids"], ref["pair_ids"])
    dt = S.U8 if m.dtype == np.uint8 else S.F32
    ws = torch.empty(S.workspace_size(m.shape, dt, 60000), dtype=torch.uint8, device="cuda")
    out, status = S.features_async(vol, sp, ws)
    assert int(status.cpu()[0]) == rc
    np.testing.assert_array_equal(out.cpu().numpy()[2:], ref["features"][2:])


def test_round_batch(S):
    """More block pairs than a wave takes of a short list: bounds tested a lane each."""
    import torch

    g = np.random.default_rng(4)
    vols, sps = [], []
    for k in range(120):
        r = float(g.uniform(4.0, 22.0))
        n = int(2 * r) + 4
        vols.append((dist((n, n, n), g.uniform(-0.5, 0.5, 3) + (n - 1) / 2.0) <= r).astype(np.uint8))
        sps.append((1.0, 1.0, 1.0) if k % 2 else tuple(g.uniform(0.9, 1.1, 3)))
    base = torch.from_numpy(np.concatenate([v.ravel() for v in vols])).cuda()
    offs = np.concatenate([[0], np.cumsum([v.size for v in vols])[:-1]])
    tab = S.roi_table(offs, [v.shape for v in vols], sps)
    say("bounds: batch of balls")
    S.set_prune(0)
    o0, s0, st0 = S.batched(base, tab, stats=True)
    S.set_prune(1)
    o1, s1, st1 = S.batched(base, tab, stats=True)
    np.testing.assert_array_equal(o1, o0)
    for r in range(len(vols)):
        np.testing.assert_array_equal(st1[r]["pair_ids"], st0[r]["pair_ids"], err_msg="ROI %d" % r)
    for r in range(0, len(vols), 17):
        ref = reference(vols[r], sps[r])
        np.testing.assert_array_equal(o1[r, 2:], ref["features"][2:])
        np.testing.assert_array_equal(st1[r]["pair_ids"], ref["pair_ids"])


def free_memory():
    import torch

    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def gpu_ball(n, r):
    import torch

    a = torch.arange(n, device="cuda", dtype=torch.float64) - (n - 1) / 2.0
    return ((a[:, None, None] ** 2 + a[None, :, None] ** 2 + a[None, None, :] ** 2) <= r * r).to(torch.uint8)


def test_the_list_of_a_ball_fits(S):
    """A ball's block pairs fit in the list that the library starts with."""
    import torch

    S.set_prune(1)
    used = []
    ball = gpu_ball(300, 148.0)
    for name, vol in (("empty", torch.zeros_like(ball)), ("ball", ball)):
        S.release()
        say("bounds: list of an %s volume" % name)
        before = free_memory()
        S.features(vol, (1.0, 1.0, 1.0))
        used.append(before - free_memory())
    assert used[1] == used[0]


def test_a_list_that_is_too_short(S):
    """One ball as 600 ROIs lists more block pairs than the first guess holds.
    Device results: nothing is read back, and the pairs are evaluated where they
    are found; with a bound of 1,130 on the dims with ids beyond 2^32, which take
    two tie passes."""
    import torch

    n, m = 600, 204
    S.set_prune(1)
    vol = gpu_ball(m, 100.0)
    sp = (1.0, 1.0, 1.0)
    f, st, _ = S.features(vol, sp, stats=True)
    S.release()
    tab = S.table_to_device(S.roi_table_ex([0] * n, [vol.shape] * n, [sp] * n))
    for side in (m, 1130):
        say("bounds: a list that is too short, side %d" % side)
        out, status = S.batched_dev(vol.view(-1), tab, n, (side, side, side))
        out, status = out.cpu().numpy(), status.cpu().numpy()
        assert np.all(status == 0)
        np.testing.assert_array_equal(out, np.tile(f, (n, 1)))
    # the host's call on the same ROIs finds the list too short and makes it longer
    before = free_memory()
    o, s, sts = S.batched(vol.view(-1), S.roi_table([0] * n, [vol.shape] * n, [sp] * n), stats=True)
    assert before - free_memory() > 100 << 20
    np.testing.assert_array_equal(o, out)
    np.testing.assert_array_equal(sts[n - 1]["pair_ids"], st["pair_ids"])
    S.release()
