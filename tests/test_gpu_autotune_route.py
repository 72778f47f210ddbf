"""GPU checks that tuning leaves the calls on the block-pair pass while pruning
is on: the choice is kernel 1 whatever was set, a cache line of the pair-pass
tiles (an older file) does not name another, and with prune = 0 the tiles are
timed, cached and used as before."""
import sys

import numpy as np
import pytest

from paper_2510_02894_amd import synth

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
    yield shape3d
    shape3d.set_tuning(8, 1024, 0, 1, prune=1)


def batch(S):
    import torch

    buf, offs, shapes, sps = synth.batched_rois(16, 8, lmin=8.0, lmax=24.0)
    return torch.from_numpy(buf).cuda(), S.roi_table(offs, shapes, sps)


@pytest.mark.parametrize("prune", [1, 2])
@pytest.mark.parametrize("before", [(8, 1024, 0, 1), (4, 64, 1, 1), (2, 64, 0, 0)])
def test_tuning_keeps_the_block_pass(S, tmp_path, prune, before):
    base, table = batch(S)
    S.set_tuning(*before, prune=prune)
    ref, _ = S.batched(base, table)
    cache = tmp_path / "tiles.txt"
    say("autotune with prune %d from %s" % (prune, before))
    best, ms = S.autotune(base, table, reps=1, cache_path=str(cache))
    assert best[3] == 1 and best[2] == 0 and ms > 0 and S.get_tuning() == best and S.get_prune() == prune
    if before[3] == 1:
        assert best[:2] == before[:2]
    # an older file: the same class without a mark of the route, won by kernel 0
    key, _, rest = cache.read_text().strip().partition(" ")
    cls = key[:-2] if key.endswith(":b") else key
    cache.write_text("%s 0 8 64 0 0.000001\n%s 0 8 64 0 0.000001\n" % (cls, key))
    S.set_tuning(*before, prune=prune)
    best, _ = S.autotune(base, table, reps=1, cache_path=str(cache))
    assert best[3] == 1 and S.get_tuning() == best
    np.testing.assert_array_equal(S.batched(base, table)[0], ref)


def test_tiles_are_tuned_where_every_pair_is_visited(S, tmp_path):
    base, table = batch(S)
    ref, _ = S.batched(base, table)
    S.set_tuning(8, 1024, 0, 1, prune=0)
    cache = tmp_path / "tiles.txt"
    say("autotune with prune 0")
    best, ms = S.autotune(base, table, reps=1, cache_path=str(cache))
    assert ms > 0 and S.get_tuning() == best
    key, kern, it, jc, bpc, _ = cache.read_text().split()
    assert (int(it), int(jc), int(bpc), int(kern)) == best and not key.endswith(":b")
    cache.write_text("%s 0 2 128 0 0.5\n" % key)
    assert S.autotune(base, table, reps=1, cache_path=str(cache)) == ((2, 128, 0, 0), 0.5)
    np.testing.assert_array_equal(S.batched(base, table)[0], ref)
