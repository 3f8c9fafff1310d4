"""Per-ring passes (extents, areas, validation) and the touching test at ring
lengths around their rows of 16 lanes and chunks of 64 vertices."""

import numpy as np
import pytest

import oracle
import paper_1208_0277_amd as sccg
from sccg_gen import concat
from tests.gpu_util import assert_exact, device_workload, run
from tests.shapes import band_ring

pytestmark = pytest.mark.gpu

SIZES = (4, 15, 16, 17, 63, 64, 65, 79, 80, 128, 129, 300)


def _stair(verts, dx=0, dy=0, step=1, width=9):
    """A staircase ring of exactly `verts` vertices (some repeated)."""
    nb = max(1, verts // 4)
    y = [dy + k for k in range(nb + 1)]
    a = [dx + step * k for k in range(nb)]
    ring = np.asarray(band_ring(y, a, [v + width for v in a]), np.int32)
    return np.repeat(ring, [1 + verts - len(ring)] + [1] * (len(ring) - 1), axis=0)


def _bad_edge(ring):
    w = np.roll(ring, -1, axis=0)
    return len(ring) < 4 or bool(np.any((ring[:, 0] != w[:, 0]) & (ring[:, 1] != w[:, 1])))


@pytest.mark.parametrize("at", [0, 1, 14, 15, 16, 62, 63, 64, 127, 128, -1])
def test_validate_finds_the_edge(at):
    """A vertex off its pixel side anywhere in a ring, and rings of three
    vertices, are found; the smallest index is reported."""
    import torch
    rings = []
    for n in SIZES:
        rings.append(_stair(n))
        bad = _stair(n)
        bad[at % n] += (3, 5) if n % 2 else (5, 3)
        rings.append(bad)
    rings.append(_stair(4)[:3])
    first = next(k for k, r in enumerate(rings) if _bad_edge(r))
    c = sccg.Context(0)
    try:
        for skip in (0, first + 1, len(rings) - 1):
            P = concat(rings[skip:])
            want = next((k for k, r in enumerate(rings[skip:]) if _bad_edge(r)), -1)
            out = c.validate_polys(sccg.DevicePolys.from_host(P.off, P.xy))
            c.sync()
            assert int(out.item()) == want
        good = concat([_stair(n) for n in SIZES])
        out = c.validate_polys(sccg.DevicePolys.from_host(good.off, good.xy))
        c.sync()
        assert int(out.item()) == -1
        assert torch.cuda.is_available()
    finally:
        c.close()


def test_ring_lengths_in_plain_mode_and_the_join():
    """Extents and areas of the per-ring pass, through PLAIN counts and the
    join's candidates; one ring too wide for an area in 32 bits."""
    import torch
    ra = [_stair(n, dx=40 * k, dy=3 * k) for k, n in enumerate(SIZES)]
    rb = [_stair(n, dx=40 * k + 2, dy=3 * k + 1, step=(k % 2)) for k, n in enumerate(reversed(SIZES))]
    ra.append(np.asarray(band_ring([-9, 40000], [-20000], [20000]), np.int32))
    rb.append(_stair(80, dx=100))
    A, B = concat(ra), concat(rb)
    idx = np.arange(len(ra), dtype=np.int32)
    eI, eU = oracle.area_pairs(A, B, idx, idx, form=oracle.ROWS)
    c = sccg.Context(0)
    try:
        I, U = run(c, device_workload(A, B, idx, idx), sccg.SCCG_PLAIN)
        assert_exact(I, U, eI, eU, "ring lengths, PLAIN")
        off = np.array([0, A.n], np.int64)
        want = oracle.join_sets(A, B, off, off)
        t = torch.from_numpy(off).cuda()
        pa, pb, so = c.join_sets(sccg.DevicePolys.from_host(A.off, A.xy), sccg.DevicePolys.from_host(B.off, B.xy), t, t, cell=512)
        c.sync()
        for g, w in zip((pa, pb, so), want):
            assert np.array_equal(g.cpu().numpy(), w)
    finally:
        c.close()


@pytest.mark.parametrize("copies", [1, 700])
def test_touching_rings_of_every_length(copies):
    """Staircases beside each other: sharing sides, a single point, or a pixel
    apart, with rings of one to five chunks; few pairs and many per wave."""
    ra, rb = [], []
    for n in SIZES:
        for m in (4, 64, 65, 129):
            h = max(1, n // 4)
            for dx, dy in ((9, 0), (9, 1), (10, 0), (9 + h - 1, h), (9 + h, h), (-9, 0), (0, h), (0, h + 1), (3, 0)):
                ra.append(_stair(n))
                rb.append(_stair(m, dx, dy))
    A, B = concat(ra), concat(rb)
    idx = np.arange(len(ra), dtype=np.int32)
    expect = oracle.relate_pairs(A, B, idx, idx)
    idx, expect = np.tile(idx, copies), np.tile(expect, copies)
    work = device_workload(A, B, idx, idx)
    c = sccg.Context(0)
    try:
        I, _ = c.area_pairs(*work)
        got = c.relate_pairs(*work, I)
        c.sync()
        assert np.array_equal(got.cpu().numpy().astype(np.uint32), expect)
    finally:
        c.close()
    assert {0, sccg.SCCG_REL_TOUCHES} < set(expect.tolist())
