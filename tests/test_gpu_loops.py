"""Rings that are not simple, which validation does not look for: their areas are
the sums of their loops, the same through every path (loops that cancel leave
|p| + |q| - I below 0)."""

import numpy as np
import pytest

import paper_1208_0277_amd as sccg
from sccg_gen import concat
from tests.gpu_util import device_workload, run

pytestmark = pytest.mark.gpu

#: an eight of two squares of side 20, one run through clockwise: no area, 800 pixels
EIGHT = np.array([(0, 0), (20, 0), (20, 40), (40, 40), (40, 20), (0, 20)], np.int32)


def _area(ring):
    x, y = ring[:, 0].astype(object), ring[:, 1].astype(object)
    return abs(int((x * np.roll(y, -1) - y * np.roll(x, -1)).sum())) // 2


@pytest.mark.parametrize("n", [200, 60000])
def test_loops_that_cancel(n):
    """Pairs whose union exceeds a tile, so that U comes from the areas: own
    tiles pair by pair and made beforehand (more pairs than rings), pair boxes
    of rings that no tile holds, the medium sweep and PLAIN."""
    wide = EIGHT * (4, 1)  # 160 wide
    rings = [EIGHT, EIGHT + (35, 25), EIGHT + (30, -30), wide, wide + (20, 10)]
    P = concat(rings)
    pa, pb = np.meshgrid(np.arange(5), np.arange(5))
    pa, pb = (np.resize(v.ravel(), n).astype(np.int32) for v in (pa, pb))
    assert all(_area(r) == 0 for r in rings)
    got = {}
    for name, mode, params in (("plain", sccg.SCCG_PLAIN, {}), ("medium", sccg.SCCG_BATCHED, {"flags": sccg.SCCG_F_NO_UNION_TILE}),
                               ("pair box", sccg.SCCG_BATCHED, {"flags": sccg.SCCG_F_NO_UNION_TILE, "sweep_pair_box": 2})):
        c = sccg.Context(0, **params)
        try:
            got[name] = run(c, device_workload(P, P, pa, pb), mode)
        finally:
            c.close()
    I, U = got["plain"]
    assert I.max() > 0 and np.array_equal(U, -I)
    for name, (i, u) in got.items():
        assert np.array_equal(i, I) and np.array_equal(u, U), name


@pytest.mark.parametrize("turns,side", [(2, 30000), (3, 32767), (40, 9000)])
def test_loops_that_add_up(turns, side):
    """A square run through several times: twice its area exceeds 32 bits.  U of
    PLAIN, and the relations of the square with as many pixels."""
    import torch
    square = np.array([(0, 0), (side, 0), (side, side), (0, side)], np.int32) - 11
    wound = np.tile(square, (turns, 1))
    small = np.array([(5, 5), (25, 5), (25, 30), (5, 30)], np.int32)
    P, Q = concat([wound, small]), concat([small, wound])
    area = _area(wound)
    assert area == turns * side * side
    inside = 500 * (turns % 2)
    work = device_workload(P, Q, np.arange(2, dtype=np.int32), np.arange(2, dtype=np.int32))
    c = sccg.Context(0)
    try:
        I, U = run(c, work, sccg.SCCG_PLAIN)
        assert I.tolist() == [inside] * 2 and U.tolist() == [area + 500 - inside] * 2
        got = c.relate_pairs(*work, torch.full((2,), area, dtype=torch.int64, device="cuda"))
        c.sync()
        assert got.tolist() == [sccg.SCCG_REL_INTERSECTS | sccg.SCCG_REL_WITHIN, sccg.SCCG_REL_INTERSECTS | sccg.SCCG_REL_CONTAINS]
    finally:
        c.close()


@pytest.mark.parametrize("side", [16384, 20000, 32767])
def test_long_rings_that_add_up(side):
    """The same of 320 and 1200 vertices in BATCHED calls."""
    square = np.array([(0, 0), (side, 0), (side, side), (0, side)], np.int32) - 11
    small = np.array([(5, 5), (25, 5), (25, 30), (5, 30)], np.int32)
    rings = [np.tile(square, (turns, 1)) for turns in (81, 300)]
    P, Q = concat(rings + [small] * 2), concat([small] * 2 + rings)
    area = [_area(r) + 500 - 500 * (len(r) // 4 % 2) for r in rings]
    idx = np.arange(4, dtype=np.int32)
    c = sccg.Context(0)
    try:
        I, U = run(c, device_workload(P, Q, idx, idx), sccg.SCCG_BATCHED)
    finally:
        c.close()
    assert I.tolist() == [500, 0] * 2 and U.tolist() == area * 2
