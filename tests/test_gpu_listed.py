"""Pairs listed for the persistent kernel, in a part per bucket and stream: few
and many of them, of every bucket, from the long pairs' teams and the medium
sweep's waves, and in a time that does not grow with one counter's atomics."""

import time

import numpy as np
import pytest

import paper_1208_0277_amd as sccg
from sccg_gen import Polys
from tests.gpu_util import assert_exact, device_workload, run

pytestmark = pytest.mark.gpu


def _combs(n, teeth, width, height):
    """n combs of teeth[k] teeth each, width x height, at (0, 0)."""
    off, rings, area = [0], [], []
    for t in teeth[:n]:
        pitch = width // (t + 1)
        pts = [(0, 0), (width, 0), (width, 9)]
        for k in range(t):  # notches from the right
            x = width - pitch * k - 3
            pts += [(x, 9), (x, height), (x - pitch // 2, height), (x - pitch // 2, 9)]
        pts += [(0, 9)]
        rings.append(np.array(pts, np.int32))
        off.append(off[-1] + len(pts))
        area.append(9 * width + t * (pitch // 2) * (height - 9))
    return Polys(np.array(off, np.int64), np.concatenate(rings)), np.array(area, np.int64)


@pytest.mark.parametrize("n", [1, 7, 8, 9, 63, 640, 5121, 20011])
@pytest.mark.parametrize("params", [{}, {"flags": sccg.SCCG_F_NO_SPLIT_QUEUE}, {"flags": sccg.SCCG_F_NO_SEP},
                                    {"min_classify_cells": 1, "heavy_verts": 300}])
def test_listed_pairs(n, params):
    """Boxes of 95 leaf tiles, rings of 28 to 812 vertices (every
    bucket): each pair with itself shifted by (0, 2)."""
    teeth = np.resize([6, 20, 45, 62, 63, 70, 120, 200], n)
    A, area = _combs(n, teeth, 1200, 300)
    B = Polys(A.off, A.xy + np.array([0, 2], np.int32))
    idx = np.arange(n, dtype=np.int32)
    pitch = 1200 // (teeth + 1)
    # the handle keeps 7 of its 9 rows and the teeth fill two of B's rows above A's handle
    inter = 7 * 1200 + teeth * (pitch // 2) * (300 - 9)
    c = sccg.Context(0, **params)
    try:
        I, U = run(c, device_workload(A, B, idx, idx), sccg.SCCG_BATCHED)
        assert_exact(I, U, inter, 2 * area - inter, f"{n} listed pairs, {params}")
    finally:
        c.close()


def test_listing_of_some_thousand_pairs():
    """5000 pairs with boxes of 90 tiles against as many with boxes of 60, which
    are counted at once: listing them took 125 us on one counter."""
    import torch
    us = {}
    for width in (760, 1100):
        A, _ = _combs(5000, np.full(5000, 2), width, 300)
        idx = np.arange(5000, dtype=np.int32)
        work = device_workload(A, A, idx, idx)
        c = sccg.Context(0, flags=sccg.SCCG_F_NO_SPLIT_QUEUE)
        try:
            out = [torch.empty(5000, dtype=torch.int64, device="cuda") for _ in range(2)]
            c.set_stats(False, stamps=True)
            best = 1e9
            for _ in range(8):
                c.area_pairs(*work, *out)
                c.sync()
                t = c.wave_times(1)  # the medium sweep, in 10 ns
                best = min(best, int(t[:, 1].max() - t[:, 0].min()) / 100)
            us[width] = best
        finally:
            c.close()
    print(f"counted {us[760]:.0f} us, listed {us[1100]:.0f} us", flush=True)
    assert us[1100] < us[760] + 50
