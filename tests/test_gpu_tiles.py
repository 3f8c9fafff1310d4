"""Pair boxes of several leaf tiles, counted in stripes of tiles: boxes around
the stripes' and the path's limits in tiles, rings around the limits of the
register chunks, against closed forms."""

import numpy as np
import pytest

import oracle
import paper_1208_0277_amd as sccg
from sccg_gen import concat
from tests.gpu_util import assert_exact, device_workload, run
from tests.shapes import band_rects, band_ring, rect_ring, rects_area, rects_inter

pytestmark = pytest.mark.gpu

#: extents of the pair box: one and two tiles, one stripe and several of a wave
#: (7 tiles) and of a team (15 tiles, 8 wide), 64 tiles and just above, flat and tall
BOXES = [(65, 64), (128, 129), (192, 130), (193, 193), (320, 320), (448, 65), (449, 64), (512, 512), (513, 512), (64, 1024),
         (130, 960), (1024, 65), (961, 250), (4096, 64), (4100, 60)]


def _band_polygon(width, height, verts, slope, dx, dy):
    """A polygon of about `verts` vertices (4 a band) that spans width x height
    exactly, its bands shifting left or right over a quarter of its width."""
    nb = max(1, min(verts // 4, height, max(1, width // 8)))
    y = [dy + height * k // nb for k in range(nb + 1)]
    span = width // 4
    at = [span * k // max(1, nb - 1) if nb > 1 else 0 for k in range(nb)]
    if slope < 0:
        at = at[::-1]
    a = [dx + v for v in at]
    b = [v + width - (span if nb > 1 else 0) for v in a]
    return y, a, b


def _padded(ring, verts):
    """The ring with vertices repeated until it has `verts`."""
    extra = verts - len(ring)
    return np.repeat(ring, [1 + extra] + [1] * (len(ring) - 1), axis=0).astype(np.int32) if extra > 0 else ring


@pytest.mark.parametrize("params", [{}, {"heavy_verts": 16}, {"min_classify_cells": 65, "min_queue_cells": 65},
                                    {"min_classify_cells": 1}, {"sweep_pair_box": 2}])
def test_boxes_of_several_tiles(params):
    ra, rb, expect = [], [], []
    for k, (w, h) in enumerate(BOXES):
        for verts in (8, 127, 192, 193, 256, 257, 1024, 1025, 2060):
            pa = _band_polygon(w + 3, h + 5, verts, 1, -7 - 11 * k, 3 * k - 40)
            pb = _band_polygon(w + 9, h + 2, verts, -1, -7 - 11 * k + 3, 3 * k - 40 + 5)
            ra.append(_padded(band_ring(*pa), verts))
            rb.append(_padded(band_ring(*pb), max(8, verts - 64 * (k % 2))))
            qa, qb = band_rects(*pa), band_rects(*pb)
            i = rects_inter(qa, qb)
            expect.append((i, rects_area(qa) + rects_area(qb) - i))
    idx = np.arange(len(ra), dtype=np.int32)
    A, B = concat(ra), concat(rb)
    assert {192, 193, 256, 257, 1024, 1025} <= set(np.diff(A.off).tolist())
    c = sccg.Context(0, **params)
    try:
        I, U = run(c, device_workload(A, B, idx, idx), sccg.SCCG_BATCHED)
    finally:
        c.close()
    assert_exact(I, U, np.array([e[0] for e in expect]), np.array([e[1] for e in expect]), f"tiles {params}")


def test_a_ring_wider_than_an_area_of_32_bits_holds():
    """A long ring above 32767 pixels a side (its area is summed in 64 bits)
    against a small one, both as p and as q."""
    wide = _band_polygon(40000, 50000, 400, 1, -20000, -20000)
    small = _band_polygon(200, 150, 300, -1, -100, 90)
    qa, qb = band_rects(*wide), band_rects(*small)
    i = rects_inter(qa, qb)
    u = rects_area(qa) + rects_area(qb) - i
    for pad in (400, 1300):
        A = concat([_padded(band_ring(*wide), pad), _padded(band_ring(*small), 300)])
        B = concat([_padded(band_ring(*small), 300), _padded(band_ring(*wide), pad)])
        idx = np.arange(2, dtype=np.int32)
        c = sccg.Context(0)
        try:
            I, U = run(c, device_workload(A, B, idx, idx), sccg.SCCG_BATCHED)
        finally:
            c.close()
        assert_exact(I, U, np.array([i, i]), np.array([u, u]), f"wide ring of {pad} vertices")


@pytest.mark.parametrize("params", [{}, {"sweep_pair_box": 2}, {"sweep_pair_box": 2, "flags": sccg.SCCG_F_NO_UNION_TILE},
                                    {"queue_chunk": 1}, {"queue_chunk": 64}])
def test_rings_and_boxes_of_the_union_sweep(params):
    """Rings around each 64-vertex chunk of the union sweep against each other,
    on union boxes (and, with the rings shifted apart, pair boxes) around 32
    and 64 columns and rows."""
    ra, rb, expect = [], [], []
    sizes = (8, 63, 64, 65, 127, 128, 129, 191, 192, 193)
    dims = (5, 31, 32, 33, 62, 63, 64, 65)
    for n, (np_, nq) in enumerate((p, q) for p in sizes for q in sizes):
        for m in range(4):
            w, h = dims[(n + m) % len(dims)], dims[(n // 3 + 3 * m) % len(dims)]
            far = 0 if m < 2 else 40  # p reaches out of the box on its left and bottom, q on its right and top
            pa = _band_polygon(w + far, h + far, np_, 1, 100 * n - far, -50 * m - far)
            pb = _band_polygon(w + far, h + far, nq, -1, 100 * n, -50 * m)
            ra.append(_padded(band_ring(*pa), np_))
            rb.append(_padded(band_ring(*pb), nq))
            qa, qb = band_rects(*pa), band_rects(*pb)
            i = rects_inter(qa, qb)
            expect.append((i, rects_area(qa) + rects_area(qb) - i))
    A, B = concat(ra), concat(rb)
    assert set(np.diff(A.off).tolist()) == set(sizes)
    idx = np.arange(len(ra), dtype=np.int32)
    c = sccg.Context(0, **params)
    try:
        I, U = run(c, device_workload(A, B, idx, idx), sccg.SCCG_BATCHED)
    finally:
        c.close()
    assert_exact(I, U, np.array([e[0] for e in expect]), np.array([e[1] for e in expect]), f"sweep {params}")


@pytest.mark.parametrize("n,params", [(60000, {}), (20000, {}), (60000, {"flags": sccg.SCCG_F_NO_UNION_TILE}),
                                      (60000, {"flags": sccg.SCCG_F_NO_SEP}), (60000, {"heavy_verts": 130})])
@pytest.mark.parametrize("base", [(0, 0), (-(1 << 30), (1 << 30) - 70), ((1 << 30) - 64, -(1 << 30))])
def test_rings_on_tiles_of_their_own(base, n, params):
    """Pairs counted from one tile per ring, with sweep_pair_box = 2, the tiles
    made pair by pair or, for many more pairs than rings, beforehand: tiles that
    many columns and rows apart, rings that just fit a tile and that do not, q
    repeated along a wave's pairs, and coordinates at the ends of their range
    (there the far rings are held back so that they stay within it)."""
    lo, hi = -(1 << 30), 1 << 30
    x0, y0 = base
    moves = (-5000, -64, -63, -62, -33, -1, 0, 1, 32, 62, 63, 64, 5000)

    def placed(w, h, dx, dy):
        return min(max(x0 + dx, lo), hi - w), min(max(y0 + dy, lo), hi - h)

    ps, qs = [], []
    for n, dx in enumerate(moves):
        for m, dy in enumerate(moves):
            w, h = ((64, 63), (33, 31), (64, 64), (65, 20), (63, 63))[(n + m) % 5]
            ps.append(((w, h) + placed(w, h, dx, dy), (8, 64, 65, 129, 192)[(2 * n + m) % 5]))
    for k, (w, h) in enumerate(((64, 63), (20, 63), (64, 64), (9, 5), (65, 63))):
        qs.append(((w, h) + placed(w, h, 0, 0), (8, 64, 65, 129, 192)[k]))

    def polygon(item, slope):
        (w, h, x, y), verts = item
        return _band_polygon(w, h, verts, slope, x, y)

    pp, qq = [polygon(t, 1) for t in ps], [polygon(t, -1) for t in qs]
    A = concat([_padded(band_ring(*g), t[1]) for g, t in zip(pp, ps)])
    B = concat([_padded(band_ring(*g), t[1]) for g, t in zip(qq, qs)])
    rp, rq = [band_rects(*g) for g in pp], [band_rects(*g) for g in qq]
    inter = np.array([[rects_inter(a, b) for b in rq] for a in rp])
    area_p, area_q = np.array([rects_area(r) for r in rp]), np.array([rects_area(r) for r in rq])
    pi = (np.arange(n) * 7 % len(ps)).astype(np.int32)
    qi = np.minimum(np.arange(n) // (n * 11 // 60), len(qs) - 1).astype(np.int32)
    qi[::5] = pi[::5] % len(qs)
    expect = inter[pi, qi]
    c = sccg.Context(0, sweep_pair_box=2, **params)
    try:
        I, U = run(c, device_workload(A, B, pi, qi), sccg.SCCG_BATCHED)
    finally:
        c.close()
    assert_exact(I, U, expect, area_p[pi] + area_q[qi] - expect, f"own tiles at {base}, {n} pairs, {params}")


def test_server_with_more_pairs_than_rings():
    """With sweep_pair_box = 2 a context pixelizes all rings of its sets first
    when pairs outnumber them; a server's set is its arena, of whose slots
    only the jobs' are valid: its calls count pair by pair."""
    rng = np.random.default_rng(5)
    rings = [rect_ring((int(x), int(y), int(x) + int(w), int(y) + int(h)))
             for x, y, w, h in zip(rng.integers(0, 60, 64), rng.integers(0, 60, 64), rng.integers(3, 50, 64), rng.integers(3, 50, 64))]
    P = concat(rings)
    pa, pb = (rng.integers(0, 64, 60000).astype(np.int32) for _ in range(2))
    wI, wU = oracle.area_pairs(P, P, np.repeat(np.arange(64, dtype=np.int32), 64), np.tile(np.arange(64, dtype=np.int32), 64))
    srv = sccg.Server(0, params={"sweep_pair_box": 2}, vertex_cap=4096, slot_cap=1024, pair_cap=1 << 17)
    try:
        for _ in range(2):
            I, U = np.zeros(60000, np.int64), np.zeros(60000, np.int64)
            srv.submit(P.off, P.xy, P.off, P.xy, pa, pb, I, U)
            done = []
            while not done:
                done = srv.poll(timeout=None)
            assert done[0]["status"] == sccg.SCCG_OK
            k = pa.astype(np.int64) * 64 + pb
            assert np.array_equal(I, wI[k]) and np.array_equal(U, wU[k])
    finally:
        srv.close()


def test_counters_with_tiles_made_beforehand():
    """The counting instances of the kernels that make and use all rings' tiles:
    the oracle's counts, and the counters of the same pairs taken in calls too
    small for that (but for the vertices XORed into slots: each ring once)."""
    rng = np.random.default_rng(11)

    def rings(n, sizes):
        out = []
        for k in range(n):
            w, h = int(rng.integers(3, 66)), int(rng.integers(3, 66))
            g = _band_polygon(w, h, sizes[k % len(sizes)], 1 if k % 2 else -1, int(rng.integers(0, 90)), int(rng.integers(0, 90)))
            out.append(_padded(band_ring(*g), sizes[k % len(sizes)]))
        return out

    A, B = concat(rings(150, (4, 12, 64, 65, 130, 192, 200))), concat(rings(90, (8, 40, 63, 128, 129, 190)))
    n = 60000
    pa, pb = np.meshgrid(np.arange(A.n), np.arange(B.n))
    every = oracle.area_pairs(A, B, pa.ravel().astype(np.int32), pb.ravel().astype(np.int32), form=oracle.ROWS)
    pick = rng.integers(0, A.n * B.n, n)
    pa, pb = pa.ravel()[pick].astype(np.int32), pb.ravel()[pick].astype(np.int32)
    dA, dB, tpa, tpb = device_workload(A, B, pa, pb)
    c = sccg.Context(0, sweep_pair_box=2)
    try:
        c.set_stats(True)
        I, U = run(c, (dA, dB, tpa, tpb), sccg.SCCG_BATCHED)
        whole = c.get_stats()
        parts = dict.fromkeys(whole, 0)
        for k in range(0, n, 20000):
            run(c, (dA, dB, tpa[k:k + 20000].contiguous(), tpb[k:k + 20000].contiguous()), sccg.SCCG_BATCHED)
            parts = {key: parts[key] + v for key, v in c.get_stats().items()}
    finally:
        c.close()
    assert_exact(I, U, every[0][pick], every[1][pick], "counters on, tiles beforehand")
    assert whole["small_pairs"] + whole["large_pairs"] + whole["empty_pairs"] == n
    verts = int((np.diff(A.off)[pa] + np.diff(B.off)[pb]).sum())
    assert whole["ring_scan_vertices"] + whole["union_tile_vertices"] == verts
    updates = "leaf_vertex_updates"
    assert 0 < whole.pop(updates) < parts.pop(updates) and whole == parts


def test_server_makes_no_tiles_of_its_arena():
    """A server's set is its arena, of whose slots only the jobs' are valid.  A
    job with more pairs than that has slots would have their tiles made: 700 MB
    of scratch, which is not taken."""
    import torch
    rng = np.random.default_rng(6)
    P = concat([rect_ring((int(x), int(y), int(x) + 20, int(y) + 30)) for x, y in rng.integers(0, 60, (64, 2))])
    n = 1_200_000
    pa, pb = (rng.integers(0, 64, n).astype(np.int32) for _ in range(2))
    both = np.arange(64, dtype=np.int32)
    wI, wU = oracle.area_pairs(P, P, np.repeat(both, 64), np.tile(both, 64))
    srv = sccg.Server(0, params={"sweep_pair_box": 2}, vertex_cap=4096, slot_cap=1 << 19, pair_cap=1 << 21)
    try:
        I, U = np.zeros(n, np.int64), np.zeros(n, np.int64)
        free = torch.cuda.mem_get_info()[0]
        srv.submit(P.off, P.xy, P.off, P.xy, pa, pb, I, U)
        done = []
        while not done:
            done = srv.poll(timeout=None)
        taken = free - torch.cuda.mem_get_info()[0]
        assert done[0]["status"] == sccg.SCCG_OK and done[0]["jobs_in_launch"] == 1
        k = pa.astype(np.int64) * 64 + pb
        assert np.array_equal(I, wI[k]) and np.array_equal(U, wU[k])
        assert taken < 200 << 20, f"{taken >> 20} MB taken"
    finally:
        srv.close()
