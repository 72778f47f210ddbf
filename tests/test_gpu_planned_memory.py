"""GPU check of the device memory that a call on a device table takes: its brick
count is a bound (every ROI as large as the largest allowed), and the staging
list and the block lists follow the vertices, not that bound."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


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
    shape3d.release()
    yield shape3d
    shape3d.release()


@pytest.mark.parametrize("graph", [False, True])
def test_memory_follows_the_vertices(S, graph):
    import torch

    n, side = 1000, 1000
    g = np.random.default_rng(2)
    m = (g.random((6, 7, 9)) < 0.4).astype(np.uint8)
    base = torch.from_numpy(m.reshape(-1)).cuda()
    sp = (1.0, 0.8, 1.2)
    tab = S.table_to_device(S.roi_table_ex([0] * n, [m.shape] * n, [sp] * n))
    ref = S.features(base.view(m.shape), sp)
    S.release()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    say("planned memory, graph %s" % graph)
    for _ in range(2):
        out, status = S.batched_dev(base, tab, n, (side, side, side), graph=graph)
        torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    assert np.all(status.cpu().numpy() == 0)
    np.testing.assert_array_equal(out.cpu().numpy(), np.tile(ref, (n, 1)))
    # bricks of 256 row-groups by 8 planes: a record, a row offset and a ROI each (under 200 bytes);
    # and lists of 2^26 vertices, half as many rows again, each with 8 bytes of key and its share
    # of block lists (under 24 bytes)
    bricks = n * (-(-(side + 1) * -(-(side + 1) // 32) // 256)) * (-(-(side + 1) // 8))
    print("bricks %d, memory %.2f GB" % (bricks, used / 1e9), flush=True)
    assert used < 200 * bricks + 24 * 1.5 * 2 ** 26
