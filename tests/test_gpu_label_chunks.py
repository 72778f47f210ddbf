"""GPU check of the label pass's 16-voxel chunks: rows shorter than a chunk, of
a chunk and around it, a first voxel at any byte of a chunk, chunks of many
labels, labels past max_label, and more chunks than one round of a workgroup's
loads.  Boxes and counts are whole numbers: equal to the oracle's."""
import ctypes

import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 50, 1), (5, 9, 3), (7, 6, 15), (4, 5, 16), (4, 5, 17), (3, 2, 31),
                                   (2, 3, 100), (70, 61, 65), (9, 300, 257)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("shift", [0, 1, 15])
def test_boxes_equal_oracle(shape, shift):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_02894_amd import shape3d as S

    S.load()
    print("[case] label chunks %s shift %d" % (shape, shift), flush=True)
    g = np.random.default_rng(sum(shape) + shift)
    # runs of labels, single voxels of others, background
    lab = np.repeat(g.integers(0, 4, -(-int(np.prod(shape)) // 11)), 11)[:int(np.prod(shape))].astype(np.uint8)
    one = g.random(lab.size) < 0.1
    lab[one] = g.integers(0, 12, int(one.sum()))
    lab = lab.reshape(shape)
    raw = torch.full((lab.size + 32,), 7, dtype=torch.uint8, device="cuda")  # other labels on both sides
    raw[shift:shift + lab.size] = torch.from_numpy(lab.reshape(-1)).cuda()
    table, counts, _ = S.label_rois(raw[shift:shift + lab.size].view(shape), (1.0, 1.0, 1.0), 9)
    rois = (S.RoiEx * 9).from_buffer_copy(table.cpu().numpy().tobytes()[:9 * ctypes.sizeof(S.RoiEx)])
    for i, e in enumerate(O.label_rois(lab, 9)):
        assert counts[i] == e["count"]
        assert (rois[i].offset, list(rois[i].dims)) == (e["offset"], [int(v) for v in e["dims"]])
