"""GPU checks of float32 volumes and gradients at addresses that are no multiple
of 4 (a volume inside a packed file or message): forward, backward, single and
batched, equal to the same call on aligned copies, and the bytes around the
gradient are left alone."""
import ctypes
import sys

import numpy as np
import pytest

from paper_2510_02894_amd import synth

pytestmark = pytest.mark.gpu

SP = (1.25, 0.7, 0.75)
GOUT = np.array([0.7, -0.3, 0.9, 0.4, -0.5, 0.6])
GUARD = 64


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


def at_offset(data, off):
    """The bytes of ``data`` on the GPU, off bytes past a 16-byte boundary, with
    guard bytes around them: the whole tensor and the data's address."""
    import torch

    raw = np.frombuffer(np.ascontiguousarray(data).tobytes(), np.uint8)
    buf = np.full(GUARD + off + raw.size + GUARD, 0xA5, np.uint8)
    buf[GUARD + off:GUARD + off + raw.size] = raw
    t = torch.from_numpy(buf).cuda()
    assert t.data_ptr() % 16 == 0
    return t, ctypes.c_void_p(t.data_ptr() + GUARD + off)


def masks():
    g = np.random.default_rng(6)
    noise = np.where(g.random((5, 9, 67)) < 0.3, 0.9 * np.ones(1), 0.2).astype(np.float32)
    return [("union", synth.soft_roi((33, 38, 41), g, 3, 4.0, 11.0, 1.0)), ("noise", noise),
            ("voxel", np.ones((1, 1, 1), np.float32))]


@pytest.mark.parametrize("off", [1, 2, 3, 6, 13])
@pytest.mark.parametrize("name,m", masks(), ids=[k for k, _ in masks()])
def test_floats_at_odd_addresses(S, name, m, off):
    import torch

    lib = S.load()
    aligned = torch.from_numpy(m).cuda()
    dims, sp = (ctypes.c_int64 * 3)(*m.shape), (ctypes.c_double * 3)(*SP)
    hold, p = at_offset(m, off)
    out = (ctypes.c_double * 6)()
    for small in (True, False):
        say("%s at %d bytes, small path %s" % (name, off, small))
        S.set_small_path(small)
        assert lib.shape3d_ex(p, S.F32, dims, sp, out, None, 0, None) == 0
        np.testing.assert_array_equal(np.array(out[:]), S.features(aligned, SP))
    feats, ref_saved = S.soft_forward(aligned, SP)
    ref = S.soft_backward(aligned, ref_saved, GOUT).cpu().numpy()
    saved = S.SoftSaved()
    assert lib.shape3d_soft_forward(p, dims, sp, out, ctypes.byref(saved), None) == 0
    np.testing.assert_array_equal(np.array(out[:]), feats)
    w = (ctypes.c_double * 6)(*GOUT)
    for goff in (0, off):
        ghold, gp = at_offset(np.full(m.shape, 7.0, np.float32), goff)
        assert lib.shape3d_soft_backward(p, ctypes.byref(saved), w, gp, None) == 0
        b = ghold.cpu().numpy()
        lo, hi = GUARD + goff, GUARD + goff + m.size * 4
        assert np.all(b[:lo] == 0xA5) and np.all(b[hi:] == 0xA5)
        np.testing.assert_array_equal(np.frombuffer(b[lo:hi].tobytes(), np.float32).reshape(m.shape), ref)


@pytest.mark.parametrize("n", [3, 12])
def test_batch_at_an_odd_address(S, n):
    """n = 12: past the ROI count from which a table gives each workgroup its ROI."""
    import torch

    g = np.random.default_rng(7)
    ms = [np.where(g.random(s) < 0.3, 0.9, 0.2).astype(np.float32) for s in g.integers(3, 12, size=(n, 3))]
    flat = np.concatenate([m.ravel() for m in ms])
    offs = np.concatenate([[0], np.cumsum([m.size for m in ms])[:-1]])
    tab = S.roi_table(offs, [m.shape for m in ms], [SP] * n)
    base = torch.from_numpy(flat).cuda()
    feats, ref_saved = S.batched_soft_forward(base, tab)
    w = np.tile(GOUT * (1, 1, 0, 0, 0, 0), (n, 1))
    ref = S.batched_soft_backward(base, tab, ref_saved, w).cpu().numpy()
    lib = S.load()
    hold, p = at_offset(flat, 3)
    out, saved = np.zeros((n, 6)), (S.SoftSaved * n)()
    d = ctypes.POINTER(ctypes.c_double)
    say("batch of %d" % n)
    assert lib.shape3d_batched_soft_forward(p, tab, n, out.ctypes.data_as(d), saved, 0, None) == 0
    np.testing.assert_array_equal(out, feats)
    ghold, gp = at_offset(np.full(flat.shape, 7.0, np.float32), 2)
    assert lib.shape3d_batched_soft_backward(p, tab, n, saved, w.ctypes.data_as(d), gp, None) == 0
    b = ghold.cpu().numpy()
    lo, hi = GUARD + 2, GUARD + 2 + flat.size * 4
    assert np.all(b[:lo] == 0xA5) and np.all(b[hi:] == 0xA5)
    np.testing.assert_array_equal(np.frombuffer(b[lo:hi].tobytes(), np.float32), ref)
