"""The filter stage over many small or empty sets: the oracle's pairs, and in a
time that does not grow with a walk over the sets (bounds of several times what
the calls take)."""

import time

import numpy as np
import pytest

import oracle
import paper_1208_0277_amd as sccg
from sccg_gen import Polys

pytestmark = pytest.mark.gpu


def _squares(off, spread=20, side=12, shift=0):
    """Squares in rows, per set, 20 px apart."""
    n = int(off[-1])
    size = np.diff(off)
    k = np.arange(n) - np.repeat(off[:-1], size)
    row = np.maximum(1, np.ceil(np.sqrt(np.repeat(size, size))).astype(np.int64))
    x, y = spread * (k % row) + shift, spread * (k // row) + shift
    v = np.stack([x, y, x + side, y, x + side, y + side, x, y + side], 1).reshape(-1, 2)
    return Polys(np.arange(n + 1, dtype=np.int64) * 4, v.astype(np.int32))


def _offsets(sizes):
    return np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)


def _layout(name):
    rng = np.random.default_rng(7)
    if name == "polygons many sets apart":
        a, b = np.zeros(1_000_000, np.int64), np.zeros(1_000_000, np.int64)
        a[rng.permutation(1_000_000)[:100]] = 1
        b[:] = a
        a[0], b[0], b[-1] = 64, 3, 2
        return a, b, 20_000
    if name == "256 sets of 16":
        return np.full(256, 16), np.full(256, 16), 250
    if name == "60,000 sets of 10 and two large ones":
        a = np.full(60_000, 10)
        a[[17, 40_000]] = 3000, 5000
        a[100:120] = 0
        b = np.full(60_000, 9)
        b[[17, 40_000]] = 500, 10
        return a, b, 1100
    if name.startswith("sets around the grids' limits"):
        n = int(name.split()[-1])
        a = rng.integers(0, 4, n)
        a[n // 2] = 5000  # more polygons than one workgroup takes
        b = rng.integers(0, 4, n)
        return a, b, 400
    if name == "a million sets":
        a = np.zeros(1_000_000, np.int64)
        a[[0, 5, 999_999]] = 64, 1000, 9
        return a, a, 2000
    raise ValueError(name)


@pytest.mark.parametrize("name", ["polygons many sets apart", "256 sets of 16", "60,000 sets of 10 and two large ones",
                                  "a million sets", *(f"sets around the grids' limits {n}" for n in (255, 256, 257, 1024, 1025, 16384, 16385))])
def test_many_sets(name):
    import torch
    sa, sb, most_us = _layout(name)
    ao, bo = _offsets(sa), _offsets(sb)
    A, B = _squares(ao), _squares(bo, shift=5)
    want = oracle.join_sets(A, B, ao, bo)
    dA, dB = sccg.DevicePolys.from_host(A.off, A.xy), sccg.DevicePolys.from_host(B.off, B.xy)
    ta, tb = torch.from_numpy(ao).cuda(), torch.from_numpy(bo).cuda()
    c = sccg.Context(0)
    try:
        best = 1e9
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            got = c.join_sets(dA, dB, ta, tb, cap=8 * A.n + 64)
            c.sync()
            best = min(best, (time.perf_counter() - t0) * 1e6)
            for g, w in zip(got, want):
                assert np.array_equal(g.cpu().numpy(), w)
    finally:
        c.close()
    print(f"{name}: {best:.0f} us", flush=True)
    assert best < most_us, f"{best:.0f} us"
