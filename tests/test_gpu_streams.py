"""GPU checks that calls on different streams and threads share the library's
workspace safely: a call whose results stay on the device returns while its
kernels still run there, and the next call, on another stream, must not touch
their buffers before they are done.  Every result equals that of the same call
made alone (both sides are deterministic, so they must be equal)."""
import sys
import threading

import numpy as np
import pytest

from paper_2510_02894_amd import synth

pytestmark = pytest.mark.gpu

SP = (1.0, 0.8, 1.2)


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


@pytest.fixture(scope="module")
def data(S):
    import torch

    lab = synth.label_map(5, (60, 150, 140), 12, 6.0, 30.0, noise=0.001)
    g = np.random.default_rng(3)
    m = synth.ellipsoid_union((90, 120, 110), synth.ellipsoid_params(g, 5, 12.0, 40.0, 30.0, 80.0)).astype(np.uint8)
    p = synth.soft_roi((40, 52, 47), g, 3, 6.0, 14.0, 1.0)
    d = {"lab": torch.from_numpy(lab).cuda(), "vol": torch.from_numpy(m).cuda(), "soft": torch.from_numpy(p).cuda()}
    table, _, maxd = S.label_rois(d["lab"], SP, 12)
    d["table"], d["max"] = table, [int(x) for x in maxd.cpu()]
    torch.cuda.synchronize()
    return d


def calls(S, d):
    """What the second stream runs: name, call, result on the host."""
    import torch

    buf, offs, shapes, sps = synth.batched_rois(20, 4, lmin=8.0, lmax=40.0)
    base = torch.from_numpy(buf).cuda()
    tab = S.roi_table(offs, shapes, sps)
    w = [1.0, 0.5, 2.0, 1.0, 1.0, 1.0]

    def soft():
        f, saved = S.soft_forward(d["soft"], SP)
        return np.concatenate([f, S.soft_backward(d["soft"], saved, w).cpu().numpy().ravel()])

    return [("features", lambda: S.features(d["vol"], SP)),
            ("shape class", lambda: S.shape_class(d["vol"], SP)),
            ("batch", lambda: S.batched(base, tab)[0]),
            ("batch replayed", lambda: S.batched(base, tab, graph=True)[0]),
            ("soft", soft),
            ("vertices", lambda: S.vertices(d["vol"], SP)[0].cpu().numpy()),
            ("device results", lambda: S.batched_dev(d["lab"].view(-1), d["table"], 12, d["max"])[0].cpu().numpy())]


@pytest.mark.parametrize("graph", [False, True])
def test_second_stream_waits(S, data, graph):
    import torch

    lab = data["lab"].view(-1)
    # (a recorded call is known by its buffers: the replays use the same ones)
    out = torch.zeros((12, 6), dtype=torch.float64, device="cuda")
    status = torch.zeros(12, dtype=torch.int32, device="cuda")

    def first():
        return S.batched_dev(lab, data["table"], 12, data["max"], graph=graph, out=out, status=status)

    first()
    torch.cuda.synchronize()
    ref = out.cpu().numpy()
    todo = calls(S, data)
    alone = [f() for _, f in todo]
    torch.cuda.synchronize()
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    for (name, f), want in zip(todo, alone):
        say("streams: device results%s, then %s" % (" replayed" if graph else "", name))
        for _ in range(3):
            out.zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(a):
                first()
            with torch.cuda.stream(b):
                got = f()
            torch.cuda.synchronize()
            np.testing.assert_array_equal(got, want, err_msg=name)
            np.testing.assert_array_equal(out.cpu().numpy(), ref, err_msg=name)


def test_threads_with_their_own_streams(S, data):
    import torch

    todo = calls(S, data)
    alone = [f() for _, f in todo]
    torch.cuda.synchronize()
    bad = []

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for i in range(2 * len(todo)):
                j = (i + k) % len(todo)
                if not np.array_equal(todo[j][1](), alone[j]):
                    bad.append((k, todo[j][0]))

    say("streams: three threads")
    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


def test_tuning_change_during_a_replay(S, data):
    """Setting the tiles drops the recorded graphs, one of which still runs."""
    import torch

    lab = data["lab"].view(-1)
    out = torch.zeros((12, 6), dtype=torch.float64, device="cuda")
    status = torch.zeros(12, dtype=torch.int32, device="cuda")
    say("streams: tiles set during a replay")
    ref = None
    for _ in range(3):
        S.batched_dev(lab, data["table"], 12, data["max"], graph=True, out=out, status=status)
        S.batched_dev(lab, data["table"], 12, data["max"], graph=True, out=out, status=status)
        S.set_tuning(*S.get_tuning())
        torch.cuda.synchronize()
        ref = out.cpu().numpy() if ref is None else ref
        np.testing.assert_array_equal(out.cpu().numpy(), ref)
