"""The filter stage's kept pairs (16 per polygon), its grown scratch and its
offsets, against the oracle."""

import numpy as np
import pytest

import oracle
import paper_1208_0277_amd as sccg
from sccg_gen import concat
from tests.shapes import rect_ring

pytestmark = pytest.mark.gpu


def _sets(seed):
    """Sets of small A squares and B rectangles that cover 0, 1, 15, 16, 17 and
    hundreds of them, empty sets, and polygons before the first and after the
    last set."""
    rng = np.random.default_rng(seed)
    ra, rb, ao, bo = [rect_ring((0, 0, 9, 9))], [rect_ring((1, 1, 5, 5))], [], []
    for s in range(12):
        ao.append(len(ra))
        bo.append(len(rb))
        if s % 5 == 3:
            continue
        ox, oy = int(rng.integers(-5000, 5000)), int(rng.integers(-5000, 5000))
        side = int(rng.integers(1, 30))
        for k in rng.permutation(side * side):
            x, y = ox + 20 * (int(k) % side), oy + 20 * (int(k) // side)
            ra.append(rect_ring((x, y, x + 12, y + 12)))
        for n in (0, 1, 5, 15, 16, 17, 18, 31, 33, 900):
            w, h = (n, 1) if n < 20 else (min(n, 30), (n + 29) // 30)
            x, y = ox + 20 * int(rng.integers(0, 3)), oy + 20 * int(rng.integers(0, 3))
            rb.append(rect_ring((x, y, x + max(1, 20 * w - 8), y + max(1, 20 * h - 8))) if n else rect_ring((x + 12, y, x + 20, y + 20)))
    ao.append(len(ra))
    bo.append(len(rb))
    ra += [rect_ring((0, 0, 40, 40))] * 3
    rb += [rect_ring((0, 0, 40, 40))] * 2
    return concat(ra), concat(rb), np.array(ao, np.int64), np.array(bo, np.int64)


@pytest.mark.parametrize("cells", [(64,), (2, 64, 500), (500, 3, 1)])
def test_pairs_kept_and_scratch_grown(cells):
    """Calls in a row on one context, cell sizes whose cells and entries exceed
    the first guess among them; each equals the oracle's join."""
    import torch
    c = sccg.Context(0)
    try:
        for seed, cell in enumerate(cells):
            A, B, ao, bo = _sets(seed)
            dA, dB = sccg.DevicePolys.from_host(A.off, A.xy), sccg.DevicePolys.from_host(B.off, B.xy)
            ta, tb = torch.from_numpy(ao).cuda(), torch.from_numpy(bo).cuda()
            want = oracle.join_sets(A, B, ao, bo)
            assert np.bincount(want[1]).max() > 100 and {15, 16, 17} & set(np.bincount(want[1]).tolist())
            for cap in (4, None, len(want[0])):  # too small at first; the default; exact
                got = c.join_sets(dA, dB, ta, tb, cell=cell, cap=cap)
                c.sync()
                for g, w in zip(got, want):
                    assert np.array_equal(g.cpu().numpy(), w)
    finally:
        c.close()


@pytest.mark.parametrize("n_pairs", [1, 255, 256, 257, 70_001, 3_000_000])
@pytest.mark.parametrize("include_zero", [False, True])
def test_jaccard_over_wave_ranges(n_pairs, include_zero):
    """Set sums when sets begin, end and lie within, on and across the waves'
    ranges of 256 or more pairs: one set, sets of 256, tiny, empty and very
    uneven ones, the first starting past pair 0."""
    import torch
    rng = np.random.default_rng(n_pairs)
    U = rng.integers(1, 5000, n_pairs).astype(np.int64)
    I = np.where(rng.random(n_pairs) < 0.4, 0, (U * rng.random(n_pairs)).astype(np.int64))
    U[rng.integers(0, n_pairs, n_pairs // 50)] = 2 ** 40
    start = min(3, n_pairs - 1)
    cuts = np.sort(rng.integers(start, n_pairs + 1, 40))
    layouts = [np.array([0, n_pairs]), np.arange(0, n_pairs + 1, 256), np.concatenate([[start], cuts, cuts[-1:], [n_pairs]]),
               np.concatenate([[0, 0], np.arange(0, min(n_pairs, 60_000) + 1, 3), [n_pairs, n_pairs]]),
               np.array([n_pairs, n_pairs])]
    tI, tU = torch.from_numpy(I).cuda(), torch.from_numpy(U).cuda()
    flags = sccg.SCCG_J_INCLUDE_ZERO if include_zero else sccg.SCCG_J_NONZERO_ONLY
    c = sccg.Context(0)
    try:
        for so in layouts:
            so = np.ascontiguousarray(so, np.int64)
            got = c.jaccard_sets(torch.from_numpy(so).cuda(), tI, tU, flags=flags)
            c.sync()
            for g, w in zip(got, oracle.jaccard_sets(so, I, U, include_zero=include_zero)):
                assert np.array_equal(g.cpu().numpy(), w)
    finally:
        c.close()


@pytest.mark.parametrize("n_a,n_b,sets", [(1, 1, 1), (4095, 300, 256), (4096, 16383, 3), (4097, 16384, 256), (4096, 16385, 257),
                                          (300, 8192, 2), (9000, 40000, 1)])
def test_small_joins(n_a, n_b, sets):
    """Around the sizes that one workgroup does by itself: the A polygons and
    sets of the grids, the counts of the scans.  B polygons are small and meet
    one or two squares of a row of A's, none, or, in empty sets, have none."""
    import torch
    rng = np.random.default_rng(n_a + n_b)
    ao = np.sort(rng.integers(0, n_a + 1, sets + 1)).astype(np.int64)
    bo = np.sort(rng.integers(0, n_b + 1, sets + 1)).astype(np.int64)
    ao[0], ao[-1], bo[0], bo[-1] = 0, n_a, 0, n_b
    row = int(np.ceil(np.sqrt(n_a / sets)))
    ra, rb = [], []
    for s in range(sets):
        for k in range(int(ao[s + 1] - ao[s])):
            x, y = 20 * (k % row) - 300, 20 * (k // row) - 77 * s
            ra.append(rect_ring((x, y, x + 12, y + 12)))
        m = max(1, int(ao[s + 1] - ao[s]))
        for k in rng.integers(0, m, int(bo[s + 1] - bo[s])):
            x, y = 20 * (int(k) % row) - 300 + int(rng.integers(-3, 18)), 20 * (int(k) // row) - 77 * s + int(rng.integers(0, 12))
            rb.append(rect_ring((x, y, x + 9, y + 7)))
    A, B = concat(ra), concat(rb)
    c = sccg.Context(0)
    try:
        dA, dB = sccg.DevicePolys.from_host(A.off, A.xy), sccg.DevicePolys.from_host(B.off, B.xy)
        want = oracle.join_sets(A, B, ao, bo)
        for _ in range(2):
            got = c.join_sets(dA, dB, torch.from_numpy(ao).cuda(), torch.from_numpy(bo).cuda())
            c.sync()
            for g, w in zip(got, want):
                assert np.array_equal(g.cpu().numpy(), w)
    finally:
        c.close()
