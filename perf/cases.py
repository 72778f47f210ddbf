"""Timing cases: the calls that programs make through the public entry points.

Masks are unions of rotated ellipsoids (lesions, organs), some of them smoothed
as a reader's contour is; soft masks are the sigmoid of a distance to such a
union, as a segmentation network's output is; label maps hold one such organ per
label.  Sizes run from the crop around a small lesion to a whole 300-slice
volume, and from one region to batches of thousands.

A case is a dict of plain values.  ``prepare`` makes what a program holds before
the call, ``run`` is one pass through the entry point, ``work`` the bytes and
operations it cannot do without, and ``exact`` its results from plain torch
FP64: the surface traced cube by cube and the diameters over vertex pairs.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2510_02894_amd import shape3d as S
from paper_2510_02894_amd import synth

DEV = "cuda"


# --------------------------------------------------------------------------
# The cases.

def listed():
    return [
        # the crop around a small lesion, one call per finding in a report: launches and latency
        dict(name="lesion", kind="single", d0=17, d1=23, d2=19, ellipsoids=1, smooth=False, shape_class=False),
        # one ordinary region (the 64^3 single ROI of the benchmark)
        dict(name="single_64", kind="single", d0=64, d1=64, d2=64, ellipsoids=1, smooth=False, shape_class=False),
        # an organ with rows of odd length, all members of the Shape class
        dict(name="organ_class", kind="single", d0=97, d1=181, d2=163, ellipsoids=3, smooth=False, shape_class=True),
        # the benchmark's large region: a whole 300-slice volume, 0.9 M vertices
        dict(name="volume", kind="single", d0=300, d1=512, d2=512, ellipsoids=20, smooth=True, shape_class=False),
        # a serving loop that leaves its results on the GPU and allocates nothing
        dict(name="async_crop", kind="async", d0=90, d1=101, d2=83, ellipsoids=2),
        # a training step on a small patch: features of a soft mask and their gradient
        dict(name="train_patch", kind="train", d0=40, d1=45, d2=39, ellipsoids=3, tau=1.0),
        # the benchmark's differentiable volume, forward and backward
        dict(name="train_256", kind="train", d0=256, d1=256, d2=256, ellipsoids=8, tau=1.0),
        # a study's regions in one eager call, the whole Shape class
        dict(name="batch_256", kind="batch", n=256, lmin=8.0, lmax=128.0, shape_class=True, graph=False),
        # the benchmark's batch: thousands of regions, recorded once and replayed
        dict(name="batch_4096", kind="batch", n=4096, lmin=8.0, lmax=128.0, shape_class=False, graph=True),
        # the benchmark's batched training step: 256 soft masks, forward and backward
        dict(name="train_batch", kind="train_batch", n=256, lmin=48.0, lmax=160.0),
        # an organ label map: boxes of all labels, then every label's features in place
        dict(name="labels", kind="labels", d0=181, d1=384, d2=384, labels=24, shape_class=True),
        # exams that start in pinned host memory, transfer and computation overlapped
        dict(name="stream", kind="stream", n=6, d0=120, d1=256, d2=251, ellipsoids=4, pinned=True,
             shape_class=False),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dims(rng, lo, hi):
    """Three extents around one size, each up to 1.4 times longer or shorter."""
    size = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return {"d%d" % k: max(6, min(hi, int(round(size * math.exp(rng.uniform(-0.34, 0.34)))))) for k in range(3)}


def draw(rng):
    kind = rng.choice(["single", "single", "volume", "async", "train", "train", "batch", "batch", "train_batch",
                       "labels", "stream"])
    if kind == "single":
        return dict(kind="single", **_dims(rng, 8, 160), ellipsoids=rng.randint(1, 6), smooth=False,
                    shape_class=rng.random() < 0.4)
    if kind == "volume":
        return dict(kind="single", d0=rng.randint(90, 300), d1=rng.randint(200, 512), d2=rng.randint(200, 512),
                    ellipsoids=rng.randint(6, 20), smooth=True, shape_class=rng.random() < 0.4)
    if kind == "async":
        return dict(kind="async", **_dims(rng, 12, 180), ellipsoids=rng.randint(1, 4))
    if kind == "train":
        return dict(kind="train", **_dims(rng, 12, 256), ellipsoids=rng.randint(2, 8), tau=rng.uniform(0.5, 2.0))
    if kind == "batch":
        return dict(kind="batch", n=_logint(rng, 2, 2048), lmin=8.0, lmax=rng.uniform(24.0, 128.0),
                    shape_class=rng.random() < 0.4, graph=rng.random() < 0.3)
    if kind == "train_batch":
        return dict(kind="train_batch", n=_logint(rng, 2, 200), lmin=rng.uniform(16.0, 48.0),
                    lmax=rng.uniform(64.0, 160.0))
    if kind == "labels":
        return dict(kind="labels", **_dims(rng, 48, 320), labels=_logint(rng, 2, 104),
                    shape_class=rng.random() < 0.5)
    return dict(kind="stream", n=rng.randint(2, 8), **_dims(rng, 48, 224), ellipsoids=rng.randint(1, 5),
                pinned=rng.random() < 0.6, shape_class=rng.random() < 0.3)


# --------------------------------------------------------------------------
# Inputs.

SPACING = (1.25, 0.7, 0.75)


def _rng(case, seed, part=0):
    words = [ord(c) for c in case["kind"]] + [int(case.get(k, 0)) for k in ("d0", "d1", "d2", "n", "labels")]
    return np.random.default_rng(np.random.SeedSequence([int(seed), int(part)] + words))


def _shape(case):
    return (case["d0"], case["d1"], case["d2"])


def _params(g, shape, n):
    """n ellipsoids that fit the array: semi-axes 0.12 to 0.4 of its extents, centres in its middle."""
    d = np.asarray(shape, dtype=np.float64)
    lo, hi = (0.25, 0.45) if n == 1 else (0.12, 0.4)
    return [(g.uniform(0.35 if n == 1 else 0.2, 0.65 if n == 1 else 0.8, size=3) * d, g.uniform(lo, hi, size=3) * d, r)
            for _, _, r in synth.ellipsoid_params(g, n, 1.0, 2.0, 0.0, 1.0)]


def _radius2(shape, centre, semi, rot, lo=(0, 0, 0), hi=None, dtype=torch.float64):
    """The normalised squared radius of an ellipsoid over the voxels [lo, hi)."""
    hi = shape if hi is None else hi
    ax = [torch.arange(lo[k], hi[k], dtype=dtype, device=DEV) - float(centre[k]) for k in range(3)]
    rr = None
    for j in range(3):
        w = [ax[k] * (float(rot[k][j]) / float(semi[j])) for k in range(3)]
        q = (w[0][:, None, None] + w[1][None, :, None]) + w[2][None, None, :]
        rr = q * q if rr is None else rr.add_(q * q)
    return rr


def _bounds(shape, centre, semi):
    reach = float(np.max(semi)) + 1.0
    lo = [max(0, int(math.floor(centre[k] - reach))) for k in range(3)]
    hi = [min(shape[k], int(math.ceil(centre[k] + reach)) + 1) for k in range(3)]
    return lo, hi


def _paint(vol, params, values):
    for (c, s, r), v in zip(params, values):
        lo, hi = _bounds(vol.shape, c, s)
        if any(b <= a for a, b in zip(lo, hi)):
            continue
        view = vol[lo[0]:hi[0], lo[1]:hi[1], lo[2]:hi[2]]
        view.masked_fill_(_radius2(vol.shape, c, s, r, lo, hi) <= 1.0, v)
    return vol


def _smoothed(vol, sigma=3.0):
    """Gaussian smoothing of the indicator, thresholded again."""
    rad = int(4 * sigma)
    w = np.exp(-0.5 * (np.arange(-rad, rad + 1) / sigma) ** 2)
    w /= w.sum()
    x = vol.float()
    for k in range(3):
        y = x * float(w[rad])
        n = x.shape[k]
        for j in range(1, rad + 1):
            if j < n:
                y.narrow(k, j, n - j).add_(x.narrow(k, 0, n - j), alpha=float(w[rad + j]))
                y.narrow(k, 0, n - j).add_(x.narrow(k, j, n - j), alpha=float(w[rad - j]))
        x = y
    return (x > 0.5).to(torch.uint8)


def _mask(case, seed, part=0):
    g = _rng(case, seed, part)
    shape = _shape(case)
    if case.get("smooth"):
        # large regions as in the benchmark: semi-axes of 20 to 90 voxels anywhere in the array
        top = min(90.0, 0.3 * min(shape))
        params = [(c * np.asarray(shape), s, r)
                  for c, s, r in synth.ellipsoid_params(g, case["ellipsoids"], 20.0, max(top, 21.0), 0.0, 1.0)]
    else:
        params = _params(g, shape, case["ellipsoids"])
    vol = _paint(torch.zeros(shape, dtype=torch.uint8, device=DEV), params, [1] * len(params))
    return _smoothed(vol) if case.get("smooth") else vol


def _soft(g, shape, n, tau):
    """sigmoid(-distance / tau) of an ellipsoid union, float32."""
    d = np.asarray(shape, dtype=np.float64)
    best = None
    for c, s, r in synth.ellipsoid_params(g, n, 1.0 / 16.0, 0.25, 0.25, 0.75):
        s = s * d
        sd = _radius2(shape, c * d, s, r, dtype=torch.float32).sqrt_().sub_(1.0).mul_(float(np.prod(s)) ** (1.0 / 3.0))
        best = sd if best is None else torch.minimum(best, sd)
    return torch.sigmoid(best.mul_(-1.0 / tau))


def _grad_weights(n, seed):
    """dL/dfeatures of a loss that weighs every feature (per row: volume ... row diameter)."""
    g = np.random.default_rng(np.random.SeedSequence([int(seed), 77]))
    w = g.uniform(0.25, 1.0, size=(n, 6)) * np.asarray([1e-3, 2e-3, 1.0, 0.5, 0.5, 0.5])
    return torch.from_numpy(w).to(DEV)


def _soft_batch(case, seed):
    g = _rng(case, seed)
    sizes = _rng(case, 0, 1)  # the regions' sizes belong to the case, their contents to the seed
    vols, shapes = [], []
    for _ in range(case["n"]):
        L = int(round(math.exp(sizes.uniform(math.log(case["lmin"]), math.log(case["lmax"])))))
        vols.append(_soft(g, (L, L, L), 8, float(g.uniform(0.5, 2.0))).reshape(-1))
        shapes.append((L, L, L))
    offsets = np.concatenate([[0], np.cumsum([v.numel() for v in vols])[:-1]])
    return torch.cat(vols), offsets, shapes, [synth.SOFT_BATCH_SPACING] * case["n"]


def _labels(case, seed):
    g = _rng(case, seed)
    shape = _shape(case)
    vol = torch.zeros(shape, dtype=torch.uint8, device=DEV)
    params = synth.ellipsoid_params(g, case["labels"], 0.03, 0.16, 0.05, 0.95)
    d = np.asarray(shape, dtype=np.float64)
    return _paint(vol, [(c * d, np.maximum(s * d, 1.5), r) for c, s, r in params], range(1, case["labels"] + 1))


def _async_vertices(shape):
    """A vertex bound for a caller's workspace: a few times the array's own surface."""
    return 6 * (shape[0] * shape[1] + shape[0] * shape[2] + shape[1] * shape[2]) + 4096


def prepare(case, seed):
    kind = case["kind"]
    if kind == "single":
        return dict(case=case, vol=_mask(case, seed))
    if kind == "async":
        ws = torch.empty(S.workspace_size(_shape(case), S.U8, _async_vertices(_shape(case))), dtype=torch.uint8,
                         device=DEV)
        return dict(case=case, vol=_mask(case, seed), ws=ws)
    if kind == "train":
        p = _soft(_rng(case, seed), _shape(case), case["ellipsoids"], case["tau"])
        return dict(case=case, p=p.requires_grad_(True), w=_grad_weights(1, seed)[0])
    if kind == "batch":
        base, offsets, shapes, spacings = synth.batched_rois_torch(case["n"], seed, case["lmin"], case["lmax"], DEV)
        return dict(case=case, base=base, table=S.roi_table(offsets, shapes, spacings))
    if kind == "train_batch":
        base, offsets, shapes, spacings = _soft_batch(case, seed)
        return dict(case=case, base=base.requires_grad_(True), table=S.roi_table(offsets, shapes, spacings),
                    w=_grad_weights(case["n"], seed))
    if kind == "labels":
        return dict(case=case, vol=_labels(case, seed))
    vols = [_mask(case, seed, i).cpu() for i in range(case["n"])]
    return dict(case=case, vols=[v.pin_memory() if case["pinned"] else v for v in vols],
                spacings=[SPACING] * case["n"])


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "single":
        f = S.shape_class if case["shape_class"] else S.features
        return dict(features=f(state["vol"], SPACING))
    if kind == "async":
        out, status = S.features_async(state["vol"], SPACING, state["ws"])
        return dict(features=out, status=status)
    if kind == "train":
        f = S.shape_features(state["p"], SPACING)
        (g,) = torch.autograd.grad(f, state["p"], grad_outputs=state["w"])
        return dict(features=f.detach(), grad=g)
    if kind == "batch":
        out, status = S.batched(state["base"], state["table"], graph=case["graph"], shape_class=case["shape_class"])
        return dict(features=out, status=status)
    if kind == "train_batch":
        f = S.batched_shape_features(state["base"], state["table"])
        (g,) = torch.autograd.grad(f, state["base"], grad_outputs=state["w"])
        return dict(features=f.detach(), grad=g)
    if kind == "labels":
        out, status = S.label_features(state["vol"], SPACING, case["labels"], shape_class=case["shape_class"])
        return dict(features=out, status=status)
    out, status = S.host_stream(state["vols"], state["spacings"], shape_class=case["shape_class"])
    return dict(features=out, status=status)


def _batch_voxels(case):
    """The expected voxel count of a batch: edges log-uniform in [lmin, lmax]."""
    lo, hi = case["lmin"], case["lmax"]
    mean = (hi ** 3 - lo ** 3) / (3.0 * math.log(hi / lo))
    # the aspects of the binary batches, log-uniform in [1/2, 2] per axis, add their mean
    aspect = (1.5 / (2.0 * math.log(2.0))) ** 3 if case["kind"] == "batch" else 1.0
    return case["n"] * mean * aspect


def work(case):
    """Every voxel is read once and compared with the threshold; features (and a
    training step's gradient, which reads the soft mask again in the sense of
    the chain rule only: counted once) are written once."""
    kind = case["kind"]
    vox = _batch_voxels(case) if kind in ("batch", "train_batch") else float(case["d0"] * case["d1"] * case["d2"])
    rows = case.get("n", 1) if kind != "labels" else case["labels"]
    if kind == "stream":
        vox *= case["n"]
    per = 8.0 if kind in ("train", "train_batch") else 1.0
    return {"bytes": vox * per + rows * 8.0 * (17 if case.get("shape_class") else 6), "flops": vox}


# --------------------------------------------------------------------------
# The same results from plain torch FP64.

def _trace_cases():
    """The triangles of each of the 256 corner patterns, as cube-edge triples.

    Corner c sits at ((c >> 2) & 1, (c >> 1) & 1, c & 1); edge 4 a + 2 o_b + o_c
    runs along axis a at offsets (o_b, o_c) along the other two, in order.  On a
    face, the crossings beside an inside corner are joined with that corner on
    the right as seen from outside (two inside corners on a diagonal stay
    apart); the joins close into loops, cut into a fan from their lowest edge.
    """
    def at(c):
        return np.array([(c >> 2) & 1, (c >> 1) & 1, c & 1])

    def edge(c, e):
        a = int(np.nonzero(at(c) != at(e))[0][0])
        o = [int(at(c)[k]) for k in range(3) if k != a]
        return 4 * a + 2 * o[0] + o[1]

    rings = []  # each face's corners, counter-clockwise seen from outside
    for f in range(3):
        g, h = (f + 1) % 3, (f + 2) % 3  # e_g x e_h = e_f
        for side in (0, 1):
            ring = []
            for dg, dh in ((0, 0), (1, 0), (1, 1), (0, 1)):
                o = [0, 0, 0]
                o[f], o[g], o[h] = side, dg, dh
                ring.append(4 * o[0] + 2 * o[1] + o[2])
            rings.append(ring if side else ring[::-1])
    table = []
    for case in range(256):
        step = {}
        for ring in rings:
            ins = [(case >> c) & 1 for c in ring]
            sides = [edge(ring[k], ring[(k + 1) % 4]) for k in range(4)]  # side k: corner k to k + 1
            enter = [k for k in range(4) if not ins[k] and ins[(k + 1) % 4]]  # into the inside, walking round
            for k in enter:
                # the run of inside corners after side k ends at the next crossing; walked
                # counter-clockwise it lies left of (its start -> its end), hence right of the reverse
                j = (k + 1) % 4
                while ins[(j + 1) % 4]:
                    j = (j + 1) % 4
                step[sides[k]] = sides[j]
        tris, seen = [], set()
        for s in sorted(step):
            if s in seen:
                continue
            loop, cur = [s], step[s]
            while cur != s:
                loop.append(cur)
                cur = step[cur]
            seen.update(loop)
            tris += [(loop[0], loop[i], loop[i + 1]) for i in range(1, len(loop) - 1)]
        table.append(tris)
    return table


_TABLE = []


def _table():
    if not _TABLE:
        tris = _trace_cases()
        out = torch.full((256, 5, 3), -1, dtype=torch.int64)
        for c, t in enumerate(tris):
            for i, tri in enumerate(t):
                out[c, i] = torch.tensor(tri)
        _TABLE.append(out.to(DEV))
    return _TABLE[0]


def _edge_vertex(P, dims2, lin, axis, spacing):
    """FP64 position of the vertex on the edges that start at padded voxel lin (flat) along axis."""
    n1, n2 = dims2[1], dims2[2]
    u = [lin // (n1 * n2) - 1, (lin // n2) % n1 - 1, lin % n2 - 1]
    stride = torch.tensor([n1 * n2, n2, 1], device=DEV)[axis]
    flat = P.reshape(-1)
    pa, pb = flat[lin], flat[lin + stride]
    t = (0.5 - pa) / (pb - pa)
    return torch.stack([(u[k].double() + torch.where(axis == k, t, torch.zeros_like(t))) * spacing[k]
                        for k in range(3)], dim=-1)


def _best_pair(pos, ids, key=None):
    """(largest squared distance, (i, j)) over the pairs (of equal key), the
    smallest (id_i, id_j) among equals; (-1, None) without a pair."""
    n = pos.shape[0]
    rows = max(64, min(4096, int(6e7 // max(n, 1))))
    best_row = []
    for a in range(0, n, rows):
        d = None
        for k in range(3):
            q = pos[a:a + rows, None, k] - pos[None, :, k]
            d = q * q if d is None else d + q * q
        if key is not None:
            d = torch.where(key[a:a + rows, None] == key[None, :], d, -1.0)
        best_row.append(d.max(dim=1).values)
    best_row = torch.cat(best_row)
    best = best_row.max()
    pairs = []
    for i in torch.nonzero(best_row == best).flatten().tolist():
        q = (pos - pos[i]) ** 2
        d = q[:, 0] + q[:, 1] + q[:, 2]
        ok = (d == best) & (ids != ids[i])
        if key is not None:
            ok &= key == key[i]
        for j in torch.nonzero(ok).flatten().tolist():
            a, b = int(ids[i]), int(ids[j])
            pairs.append((min(a, b), max(a, b), i if a < b else j, j if a < b else i))
        if len(pairs) > 256:
            pairs = [min(pairs)]
    return (float(best), min(pairs)[2:]) if pairs else (-1.0, None)


def _diameters(pos, ids, keys):
    """The maximising pair of the 3D diameter and of each axis's planes."""
    out = []
    x = pos[0]
    L2 = 0.0
    for _ in range(8):  # farthest-point sweeps: a distance that some pair has
        d = ((pos - x) ** 2).sum(dim=1)
        L2 = max(L2, float(d.max()))
        x = pos[int(d.argmax())]
    lo, hi = pos.min(dim=0).values, pos.max(dim=0).values
    reach = (torch.maximum(pos - lo, hi - pos) ** 2).sum(dim=1)
    near = torch.nonzero(reach >= L2 * (1.0 - 1e-9)).flatten()
    _, pr = _best_pair(pos[near], ids[near])
    out.append(None if pr is None else (int(near[pr[0]]), int(near[pr[1]])))
    for k in range(3):
        if pos.shape[0] <= 20000:
            out.append(_best_pair(pos, ids, keys[k])[1])
            continue
        order = torch.argsort(keys[k], stable=True)
        counts = torch.unique_consecutive(keys[k][order], return_counts=True)[1].tolist()
        best, arg, a = -1.0, None, 0
        for c in counts:
            if c > 1:
                sel = order[a:a + c]
                d, pr = _best_pair(pos[sel], ids[sel])
                if pr is not None:
                    cand = (int(sel[pr[0]]), int(sel[pr[1]]))
                    tie = arg is not None and d == best and \
                        (int(ids[cand[0]]), int(ids[cand[1]])) < (int(ids[arg[0]]), int(ids[arg[1]]))
                    if d > best or tie:
                        best, arg = d, cand
            a += c
        out.append(arg)
    return out


def _features64(vol, spacing, shape_class=False, p=None):
    """The features of one region as FP64 torch scalars.  vol: bool inside
    array; p: FP64 probabilities (with a gradient) or None for a mask."""
    dims = vol.shape
    ins = torch.nn.functional.pad(vol, (1, 1, 1, 1, 1, 1))
    P = ins.double() if p is None else torch.nn.functional.pad(p, (1, 1, 1, 1, 1, 1))
    n0, n1, n2 = ins.shape
    zero = torch.zeros(17 if shape_class else 6, dtype=torch.float64, device=DEV)
    code = torch.zeros((n0 - 1, n1 - 1, n2 - 1), dtype=torch.int16, device=DEV)
    for c in range(8):
        z, y, x = (c >> 2) & 1, (c >> 1) & 1, c & 1
        code += ins[z:n0 - 1 + z, y:n1 - 1 + y, x:n2 - 1 + x].to(torch.int16) << c
    cubes = torch.nonzero((code > 0) & (code < 255))
    if cubes.numel() == 0:
        return zero if p is None else zero + p.sum() * 0.0
    tri = _table()[code[cubes[:, 0], cubes[:, 1], cubes[:, 2]].long()]
    which, slot = torch.nonzero(tri[:, :, 0] >= 0, as_tuple=True)
    edges = tri[which, slot]                                        # [T, 3]
    start = [torch.tensor(v, device=DEV) for v in zip(*[_edge_start(e) for e in range(12)])]
    lin = ((cubes[which, 0][:, None] + start[0][edges]) * n1 + cubes[which, 1][:, None] + start[1][edges]) * n2 + \
        cubes[which, 2][:, None] + start[2][edges]
    centre = torch.tensor([0.5 * dims[k] * spacing[k] for k in range(3)], dtype=torch.float64, device=DEV)
    X = _edge_vertex(P, ins.shape, lin.reshape(-1), (edges // 4).reshape(-1), spacing).reshape(-1, 3, 3) - centre
    nrm = torch.linalg.cross(X[:, 1] - X[:, 0], X[:, 2] - X[:, 0])
    len2 = (nrm * nrm).sum(dim=1)
    area = (0.5 * torch.where(len2 > 0, torch.where(len2 > 0, len2, 1.0).sqrt(), 0.0)).sum()
    signed = ((X[:, 0] * torch.linalg.cross(X[:, 1], X[:, 2])).sum(dim=1) / 6.0).sum()
    lins, axes = [], []
    for a, (z, y, x) in enumerate(((1, 0, 0), (0, 1, 0), (0, 0, 1))):
        cross = ins[:n0 - z, :n1 - y, :n2 - x] != ins[z:, y:, x:]
        u = torch.nonzero(cross)
        lins.append((u[:, 0] * n1 + u[:, 1]) * n2 + u[:, 2])
        axes.append(torch.full_like(lins[-1], a))
    vl, va = torch.cat(lins), torch.cat(axes)
    ids = 3 * vl + va
    coords = [vl // (n1 * n2), (vl // n2) % n1, vl % n2]
    keys = [2 * coords[k] + (va == k) for k in range(3)]
    with torch.no_grad():
        arg = _diameters(_edge_vertex(P.detach(), ins.shape, vl, va, spacing), ids, keys)
    diam = []
    for pr in arg:
        if pr is None:
            diam.append(zero[0])
            continue
        sel = torch.tensor(pr, device=DEV)
        Y = _edge_vertex(P, ins.shape, vl[sel], va[sel], spacing)
        q = (Y[0] - Y[1]) ** 2
        diam.append((q[0] + q[1] + q[2]).sqrt())
    out = [signed.abs(), area] + diam
    if shape_class:
        V, A = float(signed.abs()), float(area)
        w = torch.nonzero(vol)
        n = w.shape[0]
        pts = w.double()
        pts = (pts - pts.mean(dim=0)) * torch.tensor(spacing, dtype=torch.float64, device=DEV)
        lam = torch.linalg.eigvalsh((pts.T.contiguous() @ pts / n).cpu()).clamp(min=0.0).tolist()
        k = (36.0 * math.pi * V * V) ** (1.0 / 3.0)
        more = [n * spacing[0] * spacing[1] * spacing[2], A / V, k / A, V / (math.sqrt(math.pi) * A ** 1.5),
                36.0 * math.pi * V * V / A ** 3, A / k] + [4.0 * math.sqrt(lam[i]) for i in (2, 1, 0)] + \
            [math.sqrt(lam[i] / lam[2]) if lam[2] > 0 else 0.0 for i in (1, 0)]
        out += [torch.tensor(float(v), dtype=torch.float64, device=DEV) for v in more]
    return torch.stack(out)


def _edge_start(e):
    a, rest = e // 4, [(e >> 1) & 1, e & 1]
    o = [0, 0, 0]
    for k, v in zip([k for k in range(3) if k != a], rest):
        o[k] = v
    return o


def _train64(p, spacing, w):
    q = p.detach().double().requires_grad_(True)
    f = _features64(p.detach() > 0.5, spacing, p=q)
    (g,) = torch.autograd.grad(f, q, grad_outputs=w)
    return f.detach(), g


def exact(case, seed):
    kind = case["kind"]
    # thousands of regions take longer than the whole run of the cases
    if (kind == "batch" and case["n"] > 300) or (kind == "train_batch" and case["n"] > 24):
        return None
    state = prepare(case, seed)
    cls = bool(case.get("shape_class"))
    if kind == "single":
        return dict(features=_features64(state["vol"] != 0, SPACING, cls).cpu().numpy())
    if kind == "async":
        return dict(features=_features64(state["vol"] != 0, SPACING), status=None)
    if kind == "train":
        f, g = _train64(state["p"], SPACING, state["w"])
        return dict(features=f, grad=g)
    if kind in ("batch", "train_batch"):
        feats = []
        grad = torch.zeros(state["base"].numel(), dtype=torch.float64, device=DEV) if kind == "train_batch" else None
        for r in range(case["n"]):
            R = state["table"][r]
            d = tuple(int(v) for v in R.dims)
            a, b, sp = int(R.offset), int(R.offset) + d[0] * d[1] * d[2], tuple(float(v) for v in R.spacing)
            v = state["base"].detach()[a:b].view(d)
            if kind == "batch":
                feats.append(_features64(v != 0, sp, cls))
            else:
                f, g = _train64(v, sp, state["w"][r])
                feats.append(f)
                grad[a:b] = g.reshape(-1)
        f = torch.stack(feats)
        return dict(features=f, grad=grad) if grad is not None else dict(features=f.cpu().numpy(), status=None)
    if kind == "labels":
        feats = []
        for l in range(1, case["labels"] + 1):
            v = state["vol"] == l
            w = torch.nonzero(v)
            if w.numel() == 0:
                feats.append(torch.zeros(17 if cls else 6, dtype=torch.float64, device=DEV))
                continue
            lo, hi = w.min(dim=0).values.tolist(), (w.max(dim=0).values + 1).tolist()
            feats.append(_features64(v[lo[0]:hi[0], lo[1]:hi[1], lo[2]:hi[2]].contiguous(), SPACING, cls))
        return dict(features=torch.stack(feats), status=None)
    f = [_features64(v.to(DEV) != 0, SPACING, cls).cpu().numpy() for v in state["vols"]]
    return dict(features=np.stack(f), status=None)
