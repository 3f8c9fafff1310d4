"""The work that a user of sccg has it do, as cases that can be timed and compared.

The framework counts, for pairs of rectilinear polygons, the pixels of their
intersection and union, joins two sets of polygons by their MBRs, reduces the
counts to Jaccard ratios, relates and validates polygons, and serves such
comparisons as jobs.  Every case goes through those public entry points.

Inputs are made on the GPU from the seed alone: shapes are unions of one to
four ellipses (or ten to forty, a merged blob) taken column by column and
traced along pixel sides, so that rings have the vertex counts and extents of
traced objects; the other polygon of a pair is the same shape shifted by up to
three pixels and dilated by one (which of the two is the dilated one is drawn
per pair).  The sizes are those of the repository's own workloads: objects of
at most 32 px in thousands, 10-60 px objects in hundreds of thousands, two
million with a lognormal size (median 24 px, 8-400 px, 1 % blobs), a set of
15,724 objects scaled by 1-5, and densely packed tiles.
"""

import math

import numpy as np
import torch

import paper_1208_0277_amd as sccg

#: vertices per ring of each kind of shape, on average (for `work`)
RING = {"small": 45.0, "uniform": 94.0, "mix": 72.0, "blob": 530.0}
#: leaf tiles (64 x 64 px) that the pair box of one pair covers, on average at scale 1
TILES = {"small": 1.0, "uniform": 1.0, "mix": 1.3, "blob": 16.0}
#: spacing of the objects of a densely packed tile, and candidate pairs per object there
PITCH, PAIRS_PER = 42, 4.3
FRAME = {"small": 40, "uniform": 72}


def listed():
    return [
        # one small image tile's pairs, one call: latency and launches are what counts
        {"name": "pairs_1k", "what": "pairs", "shape": "small", "pairs": 1000, "scale": 1, "stream": False, "out": False,
         "call": "area", "tuned": False},
        # a tile of a slide from its two segmentations to its Jaccard ratio: join, counts, sums
        {"name": "tile_compare", "what": "sets", "tiles": 1, "side": 1024, "op": "compare"},
        # a loop that may not allocate (a serving loop): an ordinary tile's pairs, every call on
        # the one stream, since calls share the GPU's static scratch and have to be in order
        {"name": "pairs_20k_noalloc", "what": "pairs", "shape": "uniform", "pairs": 20011, "scale": 1, "stream": False,
         "out": True, "call": "noalloc", "tuned": False},
        # the uniform workload: 200,000 pairs on a stream, into arrays that the program keeps
        {"name": "pairs_200k", "what": "pairs", "shape": "uniform", "pairs": 200000, "scale": 1, "stream": True,
         "out": True, "call": "area", "tuned": False},
        # the heavy-tailed mix of a whole slide in one call, parameters tuned for it
        {"name": "mix_2M", "what": "pairs", "shape": "mix", "pairs": 2000000, "scale": 1, "stream": True, "out": True,
         "call": "area", "tuned": True},
        # merged blobs only (tissue regions, clusters of nuclei): long rings, boxes of many leaf tiles
        {"name": "blobs_8k", "what": "pairs", "shape": "blob", "pairs": 8191, "scale": 1, "stream": False, "out": False,
         "call": "area", "tuned": False},
        # the stress set of the paper's Figure 8 at its largest scale factor: few vertices, large boxes
        {"name": "scaled_16k", "what": "pairs", "shape": "uniform", "pairs": 15724, "scale": 5, "stream": False,
         "out": False, "call": "area", "tuned": False},
        # two segmentations of sixteen dense tiles compared as a whole: join, counts, per-tile sums
        {"name": "sets_compare", "what": "sets", "tiles": 16, "side": 8192, "op": "compare"},
        # one job of a comparison service, host arrays in and host arrays out
        {"name": "serve_job", "what": "serve", "shape": "uniform", "pairs": 12007},
        # which objects contain, equal or touch which, over the candidate pairs of dense tiles
        {"name": "relate", "what": "sets", "tiles": 16, "side": 4096, "op": "relate"},
        # the per-tile sums alone, over the counts of 64 dense tiles
        {"name": "jaccard", "what": "jaccard", "sets": 64, "pairs": 9515956, "zero": False},
        # the check of a segmentation's rings before anything else is done with them
        {"name": "validate", "what": "sets", "tiles": 16, "side": 8192, "op": "validate"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small", "uniform", "uniform", "mix", "mix", "blob", "scaled", "sets", "relate", "validate",
                       "jaccard", "serve"])
    if kind in ("small", "uniform", "mix", "blob", "scaled"):
        most = {"small": 300000, "uniform": 400000, "mix": 1500000, "blob": 20000, "scaled": 30000}[kind]
        n = _log(rng, 60, most) | 1
        call = "noalloc" if n <= 262144 and rng.random() < 0.25 else "area"
        return {"what": "pairs", "shape": "uniform" if kind == "scaled" else kind, "pairs": n,
                "scale": rng.randint(2, 5) if kind == "scaled" else 1, "stream": call == "area" and rng.random() < 0.5,
                "out": call == "noalloc" or rng.random() < 0.5, "call": call, "tuned": rng.random() < 0.3}
    if kind == "sets":
        return {"what": "sets", "tiles": rng.randint(1, 14), "side": _log(rng, 500, 8000), "op": "compare"}
    if kind == "relate":
        return {"what": "sets", "tiles": rng.randint(1, 14), "side": _log(rng, 500, 4000), "op": "relate"}
    if kind == "validate":
        return {"what": "sets", "tiles": rng.randint(1, 14), "side": _log(rng, 500, 8000), "op": "validate"}
    if kind == "jaccard":
        n = _log(rng, 1000, 9000000)
        return {"what": "jaccard", "sets": _log(rng, 1, max(2, n // 50)), "pairs": n, "zero": rng.random() < 0.5}
    return {"what": "serve", "shape": rng.choice(["small", "uniform"]), "pairs": _log(rng, 1000, 60000)}


# ------------------------------------------------------------------- shapes
def _rand(g, n, lo=0.0, hi=1.0):
    return torch.rand(n, generator=g, device=g.device) * (hi - lo) + lo


def _profiles(kind, s, frame, g):
    """Column intervals [lo, hi) of shapes on canvases of side s (float tensor
    [m]) in a frame of `frame` columns, two of them left free on each side;
    lo > hi where a column holds nothing."""
    m = s.shape[0]
    xc = torch.arange(frame, device=g.device, dtype=torch.float32) - 2 + 0.5
    lo = torch.full((m, frame), 1e9, device=g.device)
    hi = torch.full((m, frame), -1e9, device=g.device)
    if kind == "blob":
        k = torch.randint(10, 41, (m,), generator=g, device=g.device)
        axes, most = (0.1, 0.25), 41
    else:
        k = torch.randint(1, 5, (m,), generator=g, device=g.device)
        axes, most = ({"small": (4 / 32, 9 / 32), "uniform": (5 / 64, 25 / 64)}.get(kind, (0.25, 0.5))), 4
    for e in range(most):
        a, b = _rand(g, m, *axes) * s, _rand(g, m, *axes) * s
        if kind == "blob" and e == 0:
            a = s / 2 - 1  # one flat ellipse through all of the canvas keeps the blob in one piece
        reach = s / 2 - a if kind == "blob" else torch.minimum(0.8 * a, s / 2 - a)
        cx = s / 2 + (2 * _rand(g, m) - 1) * reach
        cy = b + _rand(g, m) * (s - 2 * b)
        t = 1 - ((xc[None, :] - cx[:, None]) / a[:, None]) ** 2
        dy = b[:, None] * t.clamp_min(0).sqrt()
        on = (t > 0) & (e < k)[:, None]
        lo = torch.where(on, torch.minimum(lo, cy[:, None] - dy), lo)
        hi = torch.where(on, torch.maximum(hi, cy[:, None] + dy), hi)
    # a column between two covered ones is covered: the frame of the shape is one piece
    on = hi > lo
    on = (on.cumsum(1) > 0) & (on.flip(1).cumsum(1).flip(1) > 0)
    mid = s[:, None] / 2
    lo = torch.where(on, torch.where(hi > lo, lo, mid), lo)
    hi = torch.where(on, torch.maximum(hi, lo + 1), hi)
    lo = torch.where(on, (lo + 0.5).floor(), torch.full_like(lo, 1e6)).to(torch.int32)
    hi = torch.where(on, (hi + 0.5).floor(), torch.full_like(hi, -1e6)).to(torch.int32)
    hi = torch.where(on, torch.maximum(hi, lo + 1), hi)
    # columns side by side share a row: the shape is 4-connected
    lo0, hi0 = lo.clone(), hi.clone()
    for a, b in ((slice(1, None), slice(None, -1)), (slice(None, -1), slice(1, None))):
        both = on[:, a] & on[:, b]
        hi[:, a] = torch.where(both, torch.maximum(hi[:, a], lo0[:, b] + 1), hi[:, a])
        lo[:, a] = torch.where(both, torch.minimum(lo[:, a], hi0[:, b] - 1), lo[:, a])
    return lo, hi


def _dilated(lo, hi):
    """The profile dilated by one pixel (4-neighbour cross)."""
    on = hi > lo
    l, h = torch.where(on, lo - 1, lo), torch.where(on, hi + 1, hi)
    for a, b in ((slice(1, None), slice(None, -1)), (slice(None, -1), slice(1, None))):
        l[:, a] = torch.where(on[:, b], torch.minimum(l[:, a], lo[:, b]), l[:, a])
        h[:, a] = torch.where(on[:, b], torch.maximum(h[:, a], hi[:, b]), h[:, a])
    return l, h


def _rings(lo, hi, turn, x0, y0, scale):
    """Rings of the profiles, traced along pixel sides with collinear points
    left out, transposed where `turn`: (vertex counts, vertices in order)."""
    m, frame = lo.shape
    on = hi > lo
    none = torch.zeros((m, 1), dtype=torch.bool, device=lo.device)
    left = torch.cat([none, on[:, :-1]], 1)
    right = torch.cat([on[:, 1:], none], 1)

    def differs(v):
        d = v[:, 1:] != v[:, :-1]
        return torch.cat([none, d], 1), torch.cat([d, none], 1)

    x = torch.arange(frame, device=lo.device, dtype=torch.int32)[None, :].expand(m, -1)
    lp, ln = differs(lo)
    hp, hn = differs(hi)
    keep = torch.cat([torch.stack([on & (~left | lp), on & (~right | ln)], 2).reshape(m, -1),
                      torch.stack([on & (~right | hn), on & (~left | hp)], 2).flip(1).reshape(m, -1)], 1)
    vx = torch.cat([torch.stack([x, x + 1], 2).reshape(m, -1), torch.stack([x + 1, x], 2).flip(1).reshape(m, -1)], 1)
    vy = torch.cat([torch.stack([lo, lo], 2).reshape(m, -1), torch.stack([hi, hi], 2).flip(1).reshape(m, -1)], 1)
    count = keep.sum(1)
    flip = turn[:, None].expand_as(keep)[keep]
    vx, vy = vx[keep], vy[keep]
    out = torch.stack([torch.where(flip, vy, vx), torch.where(flip, vx, vy)], 1) * scale
    where = torch.repeat_interleave(torch.stack([x0, y0], 1).to(torch.int32), count, 0)
    return count, out + where


class _Csr:
    """Rings gathered in any order, laid out by shape."""

    def __init__(self, n, dev):
        self.count = torch.zeros(n, dtype=torch.int64, device=dev)
        self.parts = []

    def add(self, idx, count, xy):
        self.count[idx] = count
        self.parts.append((idx, count, xy))

    def done(self):
        off = torch.zeros(self.count.shape[0] + 1, dtype=torch.int64, device=self.count.device)
        off[1:] = self.count.cumsum(0)
        if len(self.parts) == 1:
            return off, self.parts[0][2].contiguous()
        xy = torch.empty((int(off[-1]), 2), dtype=torch.int32, device=off.device)
        for idx, count, part in self.parts:
            first = count.cumsum(0) - count
            to = torch.repeat_interleave(off[idx] - first, count) + torch.arange(part.shape[0], device=off.device)
            xy[to] = part
        return off, xy


def _overlap(lo_a, hi_a, x_a, lo_b, hi_b, x_b):
    """Pixels that profiles a and b share; their first columns stand at x_a, x_b."""
    frame = lo_a.shape[1]
    at = torch.arange(frame, device=lo_a.device)[None, :] + (x_a - x_b)[:, None]
    inside = (at >= 0) & (at < frame)
    at = at.clamp(0, frame - 1)
    part = torch.minimum(hi_a, hi_b.gather(1, at)) - torch.maximum(lo_a, lo_b.gather(1, at))
    return torch.where(inside, part.clamp_min(0), torch.zeros_like(part)).sum(1, dtype=torch.int64)


def _pixels(lo, hi):
    return (hi - lo).clamp_min(0).sum(1, dtype=torch.int64)


def _pairs(kind, n, scale, seed, dev, rings=True, truth=False):
    """Pairs (A_i, B_i): the rings of both sides, or the true counts."""
    g = torch.Generator(device=dev)
    g.manual_seed(seed * 8 + 1)
    if kind == "mix":
        side = (24 * torch.exp(0.7 * torch.randn(n, generator=g, device=dev))).round().clamp(8, 400)
        blob = _rand(g, n) < 0.01
        side = torch.where(blob, _rand(g, n, 150, 400).floor(), side)
    else:
        side = _rand(g, n, 150, 400).floor() if kind == "blob" else torch.full((n,), {"small": 32.0, "uniform": 64.0}[kind], device=dev)
        blob = torch.full((n,), kind == "blob", device=dev)
    A, B = _Csr(n, dev), _Csr(n, dev)
    I = torch.zeros(n, dtype=torch.int64, device=dev)
    U = torch.zeros(n, dtype=torch.int64, device=dev)
    per_row = 400 if kind in ("small", "uniform") else 40
    step = (72 if kind in ("small", "uniform") else 416) * scale
    for is_blob in (False, True):
        last = 0
        for top in (24, 32, 64, 128, 256, 400):
            pick = ((blob == is_blob) & (side > last) & (side <= top)).nonzero().squeeze(1)
            last = top
            for idx in pick.split(max(1024, (1 << 23) // (top + 8))):
                m = idx.shape[0]
                if m == 0:
                    continue
                s = side[idx]
                lo, hi = _profiles("blob" if is_blob else kind, s, top + 8, g)
                dlo, dhi = _dilated(lo, hi)
                swap = (_rand(g, m) < 0.5)
                alo, ahi = torch.where(swap[:, None], dlo, lo), torch.where(swap[:, None], dhi, hi)
                blo, bhi = torch.where(swap[:, None], lo, dlo), torch.where(swap[:, None], hi, dhi)
                dx = torch.randint(-3, 4, (m,), generator=g, device=dev)
                dy = torch.randint(-3, 4, (m,), generator=g, device=dev)
                turn = _rand(g, m) < 0.5
                if truth:
                    d = dy[:, None].to(torch.int32)
                    i = _overlap(alo, ahi, torch.zeros_like(dx), blo + d, bhi + d, dx)
                    I[idx] = i * scale * scale
                    U[idx] = (_pixels(alo, ahi) + _pixels(blo, bhi) - i) * scale * scale
                if rings:
                    x0, y0 = (idx % per_row) * step, (idx // per_row) * step
                    A.add(idx, *_rings(alo, ahi, turn, x0, y0, scale))
                    mx, my = torch.where(turn, dy, dx) * scale, torch.where(turn, dx, dy) * scale
                    B.add(idx, *_rings(blo, bhi, turn, x0 + mx, y0 + my, scale))
    return (A.done(), B.done()) if rings else None, I, U


def _sets(tiles, side, seed, dev, pairs):
    """Densely packed tiles: set A on a jittered lattice, set B a shifted and
    dilated copy of 85 % of it and 15 % fresh shapes at uniform places; with
    `pairs`, the candidate pairs by MBR ("all", or the first 3 n) and their
    true intersections."""
    g = torch.Generator(device=dev)
    g.manual_seed(seed * 8 + 3)
    row = max(2, side // PITCH)
    per, n = row * row, tiles * row * row
    k = torch.arange(n, device=dev)
    tile, cx, cy = k // per, (k % per) % row, (k % per) // row
    ax = cx * PITCH + torch.randint(0, 9, (n,), generator=g, device=dev)
    ay = cy * PITCH + torch.randint(0, 9, (n,), generator=g, device=dev)
    frame = FRAME["uniform"]

    def profiles(m):
        got = [_profiles("uniform", torch.full((c,), 64.0, device=dev), frame, g)
               for c in [min(1 << 17, m - j) for j in range(0, m, 1 << 17)]]
        return torch.cat([x[0] for x in got]), torch.cat([x[1] for x in got])

    alo, ahi = profiles(n)
    kept = torch.randperm(n, generator=g, device=dev)[:(85 * n) // 100].sort().values
    fresh = torch.randint(0, tiles, (max(1, (15 * n) // 100),), generator=g, device=dev).sort().values
    flo, fhi = profiles(fresh.shape[0])
    klo, khi = [torch.cat(x) for x in zip(*[_dilated(alo[j], ahi[j]) for j in kept.split(1 << 17)])]
    shift = torch.randint(-3, 4, (2, kept.shape[0]), generator=g, device=dev)
    place = torch.randint(0, max(1, row * PITCH - 40), (2, fresh.shape[0]), generator=g, device=dev)
    btile = torch.cat([tile[kept], fresh])
    order = torch.argsort(btile, stable=True)
    btile = btile[order]
    blo, bhi = torch.cat([klo, flo])[order], torch.cat([khi, fhi])[order]
    bx = torch.cat([ax[kept] + shift[0], place[0]])[order]
    by = torch.cat([ay[kept] + shift[1], place[1]])[order]
    per_row = 8

    def csr(lo, hi, t, x, y):
        c = _Csr(lo.shape[0], dev)
        gx, gy = x + (t % per_row) * side, y + (t // per_row) * side
        for idx in torch.arange(lo.shape[0], device=dev).split(1 << 17):
            c.add(idx, *_rings(lo[idx], hi[idx], torch.zeros_like(idx, dtype=torch.bool), gx[idx], gy[idx], 1))
        return c.done()

    A, B = csr(alo, ahi, tile, ax, ay), csr(blo, bhi, btile, bx, by)
    a_off = torch.arange(tiles + 1, device=dev) * per
    b_off = torch.searchsorted(btile, torch.arange(tiles + 1, device=dev))
    if not pairs:
        return A, B, a_off, b_off, None, None, None

    def mbr(lo, hi, x, y):
        on = hi > lo
        first = on.to(torch.uint8).argmax(1)
        return x + first, y + lo.amin(1), x + first + on.sum(1), y + hi.amax(1)

    a0x, a0y, a1x, a1y = mbr(alo, ahi, ax, ay)
    b0x, b0y, b1x, b1y = mbr(blo, bhi, bx, by)
    found = []
    for dj in range(6):
        for di in range(6):
            i = (b0x - 80).div(PITCH, rounding_mode="floor") + di
            j = (b0y - 80).div(PITCH, rounding_mode="floor") + dj
            ok = (i >= 0) & (i < row) & (j >= 0) & (j < row)
            a = btile * per + j.clamp(0, row - 1) * row + i.clamp(0, row - 1)
            ok &= (torch.maximum(a0x[a], b0x) < torch.minimum(a1x[a], b1x))
            ok &= (torch.maximum(a0y[a], b0y) < torch.minimum(a1y[a], b1y))
            b = ok.nonzero().squeeze(1)
            found.append(torch.stack([b, a[b]]))
    b, a = torch.cat(found, 1)
    order = torch.argsort(b * n + a)
    pa, pb = a[order], b[order]
    I = torch.zeros_like(pa)
    for c in torch.arange(pa.shape[0], device=dev).split(1 << 18):
        i, j = pa[c], pb[c]
        I[c] = _overlap(alo[i] + ay[i][:, None].int(), ahi[i] + ay[i][:, None].int(), ax[i],
                        blo[j] + by[j][:, None].int(), bhi[j] + by[j][:, None].int(), bx[j])
    U = _pixels(alo, ahi)[pa] + _pixels(blo, bhi)[pb] - I
    so = torch.searchsorted(pb, b_off)
    if pairs == "some":  # as many for every seed
        pa, pb, I, U = (v[:3 * n] for v in (pa, pb, I, U))
    return A, B, a_off, b_off, (pa.to(torch.int32), pb.to(torch.int32), so), I, U


def _counts(case, seed, dev):
    """Counts of candidate pairs and the sets they belong to."""
    g = torch.Generator(device=dev)
    g.manual_seed(seed * 8 + 5)
    n = case["pairs"]
    U = torch.randint(200, 4000, (n,), generator=g, device=dev)
    I = (U * _rand(g, n)).floor().to(torch.int64)
    I = torch.where(_rand(g, n) < 0.5, torch.zeros_like(I), torch.minimum(I, U))
    cut = torch.randint(0, n + 1, (case["sets"] - 1,), generator=g, device=dev).sort().values
    off = torch.cat([torch.zeros(1, dtype=torch.int64, device=dev), cut, torch.full((1,), n, device=dev)])
    return off, I, U


def _with_bad_ring(off, xy, seed):
    """One ring of a segmentation with a vertex off its pixel side."""
    k = int(np.random.RandomState(seed % (1 << 31)).randint(off.shape[0] - 1))
    xy = xy.clone()
    xy[int(off[k]) + 1] += torch.tensor([1, 1], dtype=torch.int32, device=xy.device)
    return xy, k


# --------------------------------------------------------------------- cases
def prepare(case, seed):
    dev = torch.device("cuda")
    if case["what"] == "jaccard":
        off, I, U = _counts(case, seed, dev)
        state = {"ctx": sccg.Context(0), "off": off, "I": I, "U": U}
    elif case["what"] == "sets":
        A, B, a_off, b_off, found, I, _ = _sets(case["tiles"], case["side"], seed, dev, "some" if case["op"] == "relate" else "")
        if case["op"] == "validate":
            A = (A[0], _with_bad_ring(*A, seed)[0])
        state = {"ctx": sccg.Context(0, sweep_pair_box=2), "A": sccg.DevicePolys(*A), "B": sccg.DevicePolys(*B),
                 "a_off": a_off, "b_off": b_off, "found": found, "I": I, "cap": 6 * (B[0].shape[0] - 1)}
        if case["op"] == "compare":  # the program keeps its counts in arrays of that capacity
            state["I"] = torch.zeros(state["cap"], dtype=torch.int64, device=dev)
            state["U"] = torch.zeros(state["cap"], dtype=torch.int64, device=dev)
    elif case["what"] == "serve":
        (A, B), _, _ = _pairs(case["shape"], case["pairs"], 1, seed, dev)
        n = case["pairs"]

        def pinned(t):
            return torch.empty(t.shape, dtype=t.dtype, pin_memory=True).copy_(t).numpy()

        idx = pinned(torch.arange(n, dtype=torch.int32, device=dev))
        state = {"server": sccg.Server(0, vertex_cap=1 << 25, slot_cap=1 << 19, pair_cap=1 << 18),
                 "A": (pinned(A[0]), pinned(A[1])), "B": (pinned(B[0]), pinned(B[1])), "pa": idx, "pb": idx.copy(),
                 "I": np.zeros(n, np.int64), "U": np.zeros(n, np.int64)}
    else:
        (A, B), _, _ = _pairs(case["shape"], case["pairs"], case["scale"], seed, dev)
        n = case["pairs"]
        # what the tuner finds for the heavy-tailed mix
        params = {"min_queue_cells": 65, "min_classify_cells": 65, "heavy_verts": 512} if case["tuned"] else {}
        stream = torch.cuda.Stream() if case["stream"] else None
        state = {"ctx": sccg.Context(0, stream=stream, **params), "A": sccg.DevicePolys(*A), "B": sccg.DevicePolys(*B),
                 "pa": torch.arange(n, dtype=torch.int32, device=dev), "pb": torch.arange(n, dtype=torch.int32, device=dev)}
        if case["out"]:
            state["I"] = torch.zeros(n, dtype=torch.int64, device=dev)
            state["U"] = torch.zeros(n, dtype=torch.int64, device=dev)
    torch.cuda.synchronize()
    state["case"] = case
    return state


def run(state):
    case = state["case"]
    if case["what"] == "serve":
        srv = state["server"]
        srv.submit(*state["A"], *state["B"], state["pa"], state["pb"], state["I"], state["U"])
        done = []
        while not done:
            done = srv.poll(timeout=None)
        r = done[0]
        return {"I": state["I"], "U": state["U"], "status": r["status"], "sum_i": r["sum_i"], "sum_u": r["sum_u"],
                "n": r["n_contrib"], "j": r["j"], "jprime": r["jprime"]}
    ctx = state["ctx"]
    if case["what"] == "jaccard":
        return ctx.jaccard_sets(state["off"], state["I"], state["U"],
                                sccg.SCCG_J_INCLUDE_ZERO if case["zero"] else sccg.SCCG_J_NONZERO_ONLY)
    if case["what"] == "sets":
        if case["op"] == "validate":
            return ctx.validate_polys(state["A"])
        if case["op"] == "relate":
            pa, pb, _ = state["found"]
            return ctx.relate_pairs(state["A"], state["B"], pa, pb, state["I"])
        A, B = state["A"], state["B"]
        pa, pb, off = ctx.join_sets(A, B, state["a_off"], state["b_off"], cap=state["cap"])
        n = pa.shape[0]
        I, U = ctx.area_pairs(A, B, pa, pb, state["I"][:n], state["U"][:n])
        return off, state["I"], state["U"], ctx.jaccard_sets(off, I, U)
    if case["call"] == "noalloc":
        return ctx.area_pairs_noalloc(state["A"], state["B"], state["pa"], state["pb"], state["I"], state["U"])
    return ctx.area_pairs(state["A"], state["B"], state["pa"], state["pb"], state.get("I"), state.get("U"))


def work(case):
    """Each ring vertex (8 B), offset (8 B), pair (8 B in, 16 B of counts out)
    once; the operations are integer ones: an extent and a crossing term per
    vertex, a scan and a count per column of each leaf tile."""
    what = case["what"]
    if what == "jaccard":
        return {"bytes": 16 * case["pairs"] + 48 * case["sets"], "flops": 12 * case["pairs"]}
    if what == "sets":
        n = case["tiles"] * max(2, case["side"] // PITCH) ** 2
        ring = RING["uniform"]
        if case["op"] == "validate":
            return {"bytes": n * (8 * ring + 8), "flops": 2 * n * ring}
        pairs, verts = PAIRS_PER * n, 2 * n * ring
        if case["op"] == "relate":
            return {"bytes": 8 * verts + 16 * n + 3 * n * 20, "flops": 10 * verts + 12 * n * ring}
        # the candidate pairs go through memory, and so do their counts
        return {"bytes": 8 * verts + 16 * n + 32 * pairs, "flops": 4 * verts + pairs * (12 + 10 * ring + 64 * 26)}
    n, ring, k = case["pairs"], RING[case["shape"]], case.get("scale", 1)
    tiles = TILES[case["shape"]] * (1 if k == 1 else max(1.0, (40 * k / 64) ** 2))
    return {"bytes": n * (2 * 8 * ring + 16 + 8 + 16), "flops": n * (2 * 12 * ring + 64 * 26 * tiles)}


def _jaccard(off, I, U, zero):
    I, U = I.double(), U.double()
    on = torch.ones_like(I) if zero else (I > 0).double()

    def per_set(v):
        c = torch.cat([torch.zeros(1, dtype=v.dtype, device=v.device), v.cumsum(0)])
        return c[off[1:]] - c[off[:-1]]

    si, su, nn = per_set(I * on), per_set(U * on), per_set(on)
    r = np.asarray((I / U.clamp_min(1) * on).cpu(), dtype=np.longdouble)
    c = np.concatenate([[np.longdouble(0)], np.cumsum(r)])
    o = off.cpu().numpy()
    jp = torch.from_numpy((c[o[1:]] - c[o[:-1]]).astype(np.float64)).to(I.device) / nn.clamp_min(1)
    return si.long(), su.long(), nn.long(), torch.where(su > 0, si / su.clamp_min(1), torch.zeros_like(su)), jp


def exact(case, seed):
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    if case["what"] == "jaccard":
        return _jaccard(*_counts(case, seed, dev), case["zero"])
    if case["what"] == "sets":
        if case["op"] == "validate":
            A = _sets(case["tiles"], case["side"], seed, dev, "")[0]
            return torch.tensor([_with_bad_ring(*A, seed)[1]])
        if case["op"] == "relate":
            return None
        _, B, _, _, (_, _, off), I, U = _sets(case["tiles"], case["side"], seed, dev, "all")
        room = torch.zeros(6 * (B[0].shape[0] - 1) - I.shape[0], dtype=torch.int64, device=dev)
        return off, torch.cat([I, room]), torch.cat([U, room]), _jaccard(off, I, U, False)
    _, I, U = _pairs(case["shape"], case["pairs"], case.get("scale", 1), seed, dev, rings=False, truth=True)
    if case["what"] == "serve":
        si, su, nn, j, jp = (float(v[0]) for v in _jaccard(torch.tensor([0, case["pairs"]], device=dev), I, U, False))
        return {"I": I, "U": U, "status": 0, "sum_i": int(si), "sum_u": int(su), "n": int(nn), "j": j, "jprime": jp}
    return I, U
