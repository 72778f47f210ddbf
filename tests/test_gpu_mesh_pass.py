"""GPU checks of the mesh pass's dense enumeration and of its loads at the sizes
where they can go wrong: bricks of more active cubes than a chunk (1,024) and
rows left over between chunks, cube rows that end at, before and after a
32-cube group and a 256-row-group brick, one voxel along an axis, rows at every
byte offset, and crops of a label map.  Counts, diameters and pairs are exact;
area and volume follow from whole-number case counts and the members of the
Shape class from whole-number moments, so they differ from the oracle's by the
rounding of its sums (fewer than 2^16 terms of 2^-53, far below 1e-10)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2510_02894_amd import synth

pytestmark = pytest.mark.gpu

SP = (1.1, 0.7, 0.9)


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


# dims and density
SHAPES = [((1, 1, 1), 1.0), ((1, 1, 31), 0.6), ((1, 1, 32), 0.6), ((7, 3, 63), 0.5), ((8, 5, 64), 0.5), ((9, 4, 33), 0.5),
          ((16, 7, 30), 0.5), ((8, 30, 31), 0.5), ((3, 255, 20), 0.3), ((3, 256, 20), 0.3), ((2, 130, 40), 0.4),
          ((40, 1, 2), 0.7), ((2, 2, 1023), 0.4), ((17, 16, 15), 1.0)]


@pytest.mark.parametrize("shape,density", SHAPES, ids=["x".join(map(str, s)) for s, _ in SHAPES])
def test_masks_at_edges(S, shape, density):
    import torch

    print("[case] mask %s" % (shape,), flush=True)
    m = (np.random.default_rng(sum(shape)).random(shape) < density).astype(np.uint8)
    m.flat[0] = m.flat[-1] = 1
    m[m > 0] = np.random.default_rng(1).integers(1, 256, int(m.sum()))  # any nonzero byte is inside
    ref = O.shape_class((m > 0).astype(np.uint8), SP)
    for off in range(0, 16, 5):  # the first voxel at any byte
        buf = torch.zeros(m.size + 16, dtype=torch.uint8, device="cuda")
        buf[off:off + m.size] = torch.from_numpy(m.reshape(-1)).cuda()
        table = S.roi_table([off], [shape], [SP])
        out, status, st = S.batched(buf, table, stats=True)
        assert (st[0]["V"], st[0]["T"]) == (ref["V"], ref["T"])
        np.testing.assert_array_equal(out[0, 2:], ref["features"][2:6])
        np.testing.assert_allclose(out[0, :2], ref["features"][:2], rtol=1e-10)
        np.testing.assert_array_equal(st[0]["pair_ids"], ref["pair_ids"])
        full, _ = S.batched(buf, table, shape_class=True)
        np.testing.assert_array_equal(full[0, :6], out[0])
        # an axis is the root of an eigenvalue, which a sum's rounding moves by
        # 2^-40 of the largest: 1e-6 of the major axis where it vanishes
        tol = np.where(np.arange(17) < 12, 0.0, np.where(np.arange(17) < 15, 1e-6 * max(ref["features"][12], full[0, 12]), 1e-6))
        assert np.all(np.abs(full[0] - ref["features"]) <= 1e-9 * np.abs(ref["features"]) + tol)


@pytest.mark.parametrize("shift", [0, 1, 3])
def test_label_crops(S, shift):
    import torch

    print("[case] label crops %d" % shift, flush=True)
    lab = synth.label_map(5, (20, 45, 71), 4, 4.0, 14.0, noise=0.02)
    dev = torch.from_numpy(lab).cuda()
    lo, shape = (1, 2, 4 + shift), (17, 40, 61)
    off = (lo[0] * 45 + lo[1]) * 71 + lo[2]
    labels = [1, 2, 3, 4, 0]
    tab = S.roi_table_ex([off] * 5, [shape] * 5, [SP] * 5, strides=[(45 * 71, 71)] * 5, labels=labels)
    out, status = S.batched_dev(dev.view(-1), S.table_to_device(tab), 5, shape)
    out = out.cpu().numpy()
    crop = lab[lo[0]:lo[0] + shape[0], lo[1]:lo[1] + shape[1], lo[2]:lo[2] + shape[2]]
    for r, l in enumerate(labels):
        ref = O.shape3d((crop == l if l else crop != 0).astype(np.uint8), SP)
        np.testing.assert_array_equal(out[r, 2:], ref["features"][2:], err_msg="label %d" % l)
        np.testing.assert_allclose(out[r, :2], ref["features"][:2], rtol=1e-10)
