"""The per-ring passes over many short rings (four lanes a ring, from 2^17 rings
of few vertices on average on): lengths around their steps, a few long and wide
rings among them, averages on both sides of the change."""

import time

import numpy as np
import pytest

import oracle
import paper_1208_0277_amd as sccg
from sccg_gen import Polys, concat
from tests.shapes import band_ring

pytestmark = pytest.mark.gpu

MANY = 1 << 17
SIZES = (4, 5, 7, 8, 15, 16, 17, 31, 32, 33, 48, 49)


def _ring(verts, at, width=9, step=1):
    """A staircase of `verts` vertices, its corner at (at, -at % 977)."""
    nb = max(1, verts // 4)
    y = [-(at % 977) + k for k in range(nb + 1)]
    a = [at + step * k for k in range(nb)]
    ring = np.asarray(band_ring(y, a, [v + width for v in a]), np.int32)
    return np.repeat(ring, [1 + verts - len(ring)] + [1] * (len(ring) - 1), axis=0)


def _area(ring):
    x, y = ring[:, 0].astype(np.int64), ring[:, 1].astype(np.int64)
    return abs(int((x * np.roll(y, -1) - y * np.roll(x, -1)).sum())) // 2


def _tiled(rings, n):
    """n rings, `rings` over and over: the polygons, and which ring each is."""
    which = np.arange(n) % len(rings)
    one = concat(rings)
    size = np.diff(one.off)[which]
    off = np.concatenate([[0], np.cumsum(size)]).astype(np.int64)
    reps = -(-n // len(rings))
    return Polys(off, np.tile(one.xy, (reps, 1))[:off[-1]].copy()), which


def _dev(P):
    return sccg.DevicePolys.from_host(P.off, P.xy)


@pytest.mark.parametrize("most", [16, 33, 49])
@pytest.mark.parametrize("n", [MANY - 1, MANY, MANY + 77])
def test_validate_many_short_rings(n, most):
    rings = [_ring(v, 3 * k) for k, v in enumerate(s for s in SIZES if s <= most)]
    P, which = _tiled(rings, n)
    size = np.diff(P.off)
    c = sccg.Context(0)
    try:
        rng = np.random.default_rng(n + most)
        picks = [[n - 1], [0, n - 1], *([int(k)] for k in rng.integers(0, n, 6))]
        for bad in [[]] + picks:
            xy = P.xy.copy()
            for k in bad:  # a vertex off its pixel side, anywhere in the ring
                xy[P.off[k] + rng.integers(0, size[k])] += (1000, 2000)
            out = c.validate_polys(_dev(Polys(P.off, xy)))
            c.sync()
            assert int(out.item()) == min(bad, default=-1), (bad, size[bad])
        # a ring of three vertices among them
        off = P.off.copy()
        off[which.size // 2 + 1:] -= size[which.size // 2] - 3
        xy = np.concatenate([P.xy[:P.off[n // 2] + 3], P.xy[P.off[n // 2 + 1]:]])
        out = c.validate_polys(_dev(Polys(off, xy)))
        c.sync()
        assert int(out.item()) == n // 2
    finally:
        c.close()


@pytest.mark.parametrize("sizes", [SIZES[:5], SIZES, SIZES[8:] + (64, 65, 80)])
def test_extents_and_areas_of_many_short_rings(sizes):
    """Areas through the relations of every ring with itself (its area as their
    count: equal; one more: intersecting), among them an empty ring, one of 300
    vertices and one too wide for an area in 32 bits; extents through the join
    of sets of nine."""
    import torch
    rings = [_ring(v, 5 * k) for k, v in enumerate(sizes)] + [
        _ring(300, 11), np.asarray(band_ring([-9, 40000], [-20000], [20000]), np.int32), np.zeros((0, 2), np.int32)]
    if len(sizes) < 8:
        rings = rings[:-2] * 40 + rings  # the 300 vertices stay few
    n = MANY // 2 + 9
    P, which = _tiled(rings, n)
    area = np.array([_area(r) if len(r) else 0 for r in rings], np.int64)[which]
    dP = _dev(P)
    c = sccg.Context(0)
    try:
        i = torch.arange(n, dtype=torch.int32, device="cuda")
        every = sccg.SCCG_REL_INTERSECTS | sccg.SCCG_REL_CONTAINS | sccg.SCCG_REL_WITHIN | sccg.SCCG_REL_EQUALS
        for more in (0, 1):
            got = c.relate_pairs(dP, dP, i, i, torch.from_numpy(area + more).cuda())
            c.sync()
            want = np.where(area + more > 0, every if more == 0 else sccg.SCCG_REL_INTERSECTS, 0)
            assert np.array_equal(got.cpu().numpy(), want.astype(np.int32))
        so = np.arange(0, n + 1, 9, dtype=np.int64)
        so[-1] = n
        t = torch.from_numpy(so).cuda()
        got = c.join_sets(dP, dP, t, t, cell=4096, cap=12 * n)
        c.sync()
        for g, w in zip(got, oracle.join_sets(P, P, so, so)):
            assert np.array_equal(g.cpu().numpy(), w)
    finally:
        c.close()


def test_rectangles_validate_in_half_the_time_of_outlines():
    """A million rectangles against a million rings of 40 vertices (a third of
    the time; more than two thirds when each takes a row)."""
    import torch
    us = {}
    for verts in (4, 40):
        P, _ = _tiled([_ring(verts, 0)], 1_000_000)
        d, c = _dev(P), sccg.Context(0)
        try:
            c.validate_polys(d)
            torch.cuda.synchronize()
            best = 1e9
            for _ in range(5):
                t0 = time.perf_counter()
                for _ in range(40):
                    c.validate_polys(d)
                torch.cuda.synchronize()
                best = min(best, (time.perf_counter() - t0) / 40 * 1e6)
            us[verts] = best
        finally:
            c.close()
    print(f"rectangles {us[4]:.0f} us, 40 vertices {us[40]:.0f} us", flush=True)
    assert us[4] < 0.5 * us[40]
